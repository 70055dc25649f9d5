// Three-level hybrid Schwarz multigrid (HSMG) preconditioner of the pressure
// Poisson operator (Sec. 3: the pressure GMRES is preconditioned by a
// three-level HSMG with a coarse-grid solve).  Periodic box of equal
// elements; levels of order N (fine), N/2 (middle) and 1 (coarse):
//
//   M^{-1} r = S_f r + P_fm ( S_m r_m + P_mc A_c^+ R_cm r_m ),  r_m = R_mf r
//
// S_l: additive Schwarz over element subdomains; the local problem is the
// element's separable stiffness, extended by one linear segment to a zero
// Dirichlet node on each side, solved by fast diagonalisation
// (u = S3 diag(1/(lx_i + ly_j + lz_k)) S3^T r); the local solutions of all
// copies of a node are summed and divided by their number.
// P: tensor-product Lagrange interpolation between the levels' GLL points;
// R = P^T in the unique-node inner product (R r = dssum(P_e^T (r / mult))).
// A_c^+: exact solve of the order-1 operator off the constant mode, by fast
// diagonalisation on the nx ny nz corner nodes.
//
// One apply = 5 launches (7 for a large coarse grid), every one gated per request:
//   hs_down   (fine FDM solve -> F_HSF; fine->middle restriction -> F_HRM)
//   hs_mid    (sum copies of F_HRM; middle FDM -> F_HSM; middle->coarse -> F_HC8)
//   hs_csmall (coarse rhs on unique corner nodes, S^T, eigenvalue scaling, S
//             -> F_HCB), or for large grids
//   hs_cxy, hs_cz, hs_cxy (coarse rhs, S^T along x and y -> F_HCB; z with the
//             scaling and S along z -> F_HCA; S along x and y -> F_HCB)
//   hs_midup  (z_m = summed F_HSM / count + trilinear coarse correction -> F_HZM)
//   hs_up     (z = summed F_HSF / count + J3 z_m -> F_HZ and Z_J of F_HZS)
// It runs in the Arnoldi steps only: the cycle end forms x += sum_j y_j Z_j
// from the kept Z_j (M is linear, so this is x += M^{-1} V y).
// The copy sums use index arithmetic on the periodic box in an order shared
// by all copies of a node, so every copy receives the identical value.
#include "k_lines.h"

namespace semk {

// the copies of 1D index i of element column ex (n elements, order N):
// (element, index) pairs, left element first
struct Cand {
    int e[2], i[2], n;
};
__device__ __forceinline__ Cand cand(int i, int ex, int n, int N)
{
    Cand c;
    if (i == 0) { c.e[0] = ex == 0 ? n - 1 : ex - 1; c.i[0] = N; c.e[1] = ex; c.i[1] = 0; c.n = 2; }
    else if (i == N) { c.e[0] = ex; c.i[0] = N; c.e[1] = ex + 1 == n ? 0 : ex + 1; c.i[1] = 0; c.n = 2; }
    else { c.e[0] = ex; c.i[0] = i; c.e[1] = ex; c.i[1] = i; c.n = 1; }
    return c;
}

// v[k] = sum of the copies of node (i,j,k) of element (ex,ey,ez) in the
// [E][L^3] field f, lower element first along z, then y, then x; returns
// 1 / (copies in a layer of elements), exact.  The one to four (y, x) neighbour
// columns are read one after the other, the points of one together (a loop over
// the copies of a point waits for each).  At k = 0 and N they add the lower
// layer's copies first, the upper's follow.
template <int L>
__device__ __forceinline__ double copies(const SEM_GLOBAL double* f, const int* nel, int ex, int ey, int ez,
                                         int i, int j, double (&v)[L])
{
    constexpr int N = L - 1, L2 = L * L, L3 = L2 * L;
    const int nx = nel[0], ny = nel[1], nz = nel[2], nxy = nx * ny;
    const Cand cx = cand(i, ex, nx, N), cy = cand(j, ey, ny, N);
    const int zd = nxy * (ez == 0 ? nz - 1 : ez - 1), zu = nxy * (ez + 1 == nz ? 0 : ez + 1);
    double w0[4], wN[4];
#pragma unroll
    for (int k = 0; k < L; ++k) v[k] = 0.0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const int b = h >> 1, a = h & 1;
        w0[h] = wN[h] = 0.0;      // a +0 changes no bit of a sum that began with one
        if (b < cy.n && a < cx.n) {
            const int exy = cx.e[a] + nx * cy.e[b], in = cx.i[a] + L * cy.i[b];
            const SEM_GLOBAL double* c = f + (long long)(exy + nxy * ez) * L3 + in;
            const double d0 = f[(long long)(exy + zd) * L3 + in + L2 * N];
            wN[h] = f[(long long)(exy + zu) * L3 + in];
            double x[L];
#pragma unroll
            for (int k = 0; k < L; ++k) x[k] = c[L2 * k];
            w0[h] = x[0];
            x[0] = d0;
#pragma unroll
            for (int k = 0; k < L; ++k) v[k] += x[k];
        }
    }
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        v[0] += w0[h];
        v[N] += wN[h];
    }
    return (cx.n == 2 ? 0.5 : 1.0) * (cy.n == 2 ? 0.5 : 1.0);
}

__device__ __forceinline__ double inv_mult(int i, int j, int k, int N)
{
    return (i == 0 || i == N ? 0.5 : 1.0) * (j == 0 || j == N ? 0.5 : 1.0) * (k == 0 || k == N ? 0.5 : 1.0);
}

// Fast-diagonalisation solve of one element at order L - 1.  Thread (i, j)
// of L*L holds column v[k] of the input and receives the column of the
// solution.  S[c][i*L+k] = component i of eigenvector k, lam[c][k].
// sA, sB: L^3 LDS scratch; one barrier before the first write.
template <int L>
__device__ __forceinline__ void fdm_solve(double (&v)[L], const double* sS, const double* sLam, double* sA,
                                          double* sB, int i, int j)
{
    constexpr int L2 = L * L;
    const double* Sx = sS;
    const double* Sy = sS + L2;
    const double* Sz = sS + 2 * L2;
    double w[L];
    // forward, x: w[k] = sum_a Sx[a][i] v(a, j, k)
    __syncthreads();
#pragma unroll
    for (int k = 0; k < L; ++k) sA[k * L2 + j * L + i] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < L; ++k) {
        double s = 0.0;
#pragma unroll
        for (int a = 0; a < L; ++a) s += Sx[a * L + i] * sA[k * L2 + j * L + a];
        w[k] = s;
    }
    // forward, y
#pragma unroll
    for (int k = 0; k < L; ++k) sB[k * L2 + j * L + i] = w[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < L; ++k) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < L; ++b) s += Sy[b * L + j] * sB[k * L2 + b * L + i];
        v[k] = s;
    }
    // forward z, scaling, inverse z (in registers)
    const double lij = sLam[i] + sLam[L + j];
#pragma unroll
    for (int k = 0; k < L; ++k) {
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < L; ++c) s += Sz[c * L + k] * v[c];
        w[k] = s / (lij + sLam[2 * L + k]);
    }
#pragma unroll
    for (int k = 0; k < L; ++k) {
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < L; ++c) s += Sz[k * L + c] * w[c];
        v[k] = s;
    }
    // inverse y (sA was last read before the barrier above)
#pragma unroll
    for (int k = 0; k < L; ++k) sA[k * L2 + j * L + i] = v[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < L; ++k) {
        double s = 0.0;
#pragma unroll
        for (int b = 0; b < L; ++b) s += Sy[j * L + b] * sA[k * L2 + b * L + i];
        w[k] = s;
    }
    // inverse x
#pragma unroll
    for (int k = 0; k < L; ++k) sB[k * L2 + j * L + i] = w[k];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < L; ++k) {
        double s = 0.0;
#pragma unroll
        for (int a = 0; a < L; ++a) s += Sx[i * L + a] * sB[k * L2 + j * L + a];
        v[k] = s;
    }
}

__device__ __forceinline__ void elem_xyz(int e, const int* nel, int& ex, int& ey, int& ez)
{
    ex = e % nel[0];
    const int r = e / nel[0];
    ey = r % nel[1];
    ez = r / nel[1];
}

// ---------------------------------------------------------------- fine level, down
// prefix over fine-level blocks (hs_fepb elements each), an argument of these
// two kernels alone: every launch copies its arguments
struct HsFine {
    int p[SEM_MAXB + 1];
};
// r = s_J V_J (basis storage TB)
//
// Bound by memory (V in, the local solution out, a quarter for r_m).  Every stage
// is a contraction of whole lines in place: sA[k][j][i] in rows of an odd pitch,
// sC[k][j][a] the restriction's part, which the x, y and z stages take along with
// the solve's.  Two LDS reads per multiply-add had cost, us a launch: fp64 20^3,
// LX = 10 138 -> 46 (28 for the bytes), 32^3, LX = 8 137 -> under 65; 12 requests
// of 4..9^3, LX = 6 14.1 -> 9.4.
template <int LX, typename TB>
__global__ void __launch_bounds__(hs_fepb(LX) * LX * LX) hs_down_kernel(Batch bt, HsFine hf, int gate)
{
    constexpr int LM = hs_lxm(LX), L2 = LX * LX, L3 = L2 * LX, N = LX - 1, P = LX | 1, PM = LM | 1;
    constexpr int EP = hs_fepb(LX);
    __shared__ double sAs[EP * L2 * P], sCs[EP * L2 * PM];
    const int g = blockIdx.x;
    const int ri = find_req(hf.p, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    if (!gate_ok(R, gate)) return;
    const int el = EP > 1 ? threadIdx.x / L2 : 0, t = threadIdx.x - el * L2, q = t % LX, p = t / LX;
    const int e0 = (g - hf.p[ri]) * EP + el;
    const bool live = e0 < R->E;
    const int e = live ? e0 : 0;   // lanes past the last element work on element 0 and store nothing
    double* const sA = sAs + el * L2 * P;
    double* const sC = sCs + el * L2 * PM;
    const HsOff o = hs_off(LX, R->nel);
    const double* tb = (const double*)gfield<double>(R, F_HST);
    Rows<LX, double> Sx, Sy, Sz;
    Rows<LM, double> Jm;
    Sx.set(tb + o.Sf);
    Sy.set(tb + o.Sf + L2);
    Sz.set(tb + o.Sf + 2 * L2);
    Jm.set(tb + o.J);
    const double lij = gp(tb)[o.Lf + q] + gp(tb)[o.Lf + LX + p];   // of column (i, j) = (q, p)

    const long long base = (long long)e * L3;
    {
        const int J = gp(R->I)[I_GJ];
        const double sc = gp(R->S)[S_GVS + J];
        const SEM_GLOBAL TB* V = gfield<TB>(R, F_V) + (long long)J * R->np;
        double v[LX];
#pragma unroll
        for (int k = 0; k < LX; ++k) v[k] = sc * (double)V[base + t + L2 * k];
#pragma unroll
        for (int k = 0; k < LX; ++k) sA[(k * LX + p) * P + q] = v[k];
    }
    block_sync_lds();
    {   // x: line (j, k) = (q, p)
        double* x = sA + t * P;
        double v[LX], y[LX], m[LM];
#pragma unroll
        for (int a = 0; a < LX; ++a) v[a] = x[a];
        rows_down<LX>(Sx, [&](int a) { return v[a]; }, y);
#pragma unroll
        for (int a = 0; a < LX; ++a) x[a] = y[a];
        rows_down<LX>(Jm, [&](int a) { return v[a] * inv_mult(a, q, p, N); }, m);
#pragma unroll
        for (int a = 0; a < LM; ++a) sC[t * PM + a] = m[a];
    }
    block_sync_lds();
    {   // y: line (i, k) = (q, p); of the restriction (a, k), a = t % LM
        double* x = sA + p * LX * P + q;
        double y[LX], m[LM];
        rows_down<LX>(Sy, [&](int b) { return x[b * P]; }, y);
#pragma unroll
        for (int b = 0; b < LX; ++b) x[b * P] = y[b];
        if (t < LM * LX) {
            double* c = sC + (t / LM) * LX * PM + t % LM;
            rows_down<LX>(Jm, [&](int b) { return c[b * PM]; }, m);
#pragma unroll
            for (int b = 0; b < LM; ++b) c[b * PM] = m[b];
        }
    }
    block_sync_lds();
    {   // z, the scaling and z back: column (i, j); of the restriction (a, b)
        double* x = sA + p * P + q;
        double y[LX];
        rows_down<LX>(Sz, [&](int c) { return x[c * LX * P]; }, y);
#pragma unroll
        for (int k = 0; k < LX; ++k) y[k] = y[k] / (lij + gp(tb)[o.Lf + 2 * LX + k]);
        rows_up<LX>(Sz, y, [&](int k, double v) { x[k * LX * P] = v; });
        if (t < LM * LM) {
            const double* c = sC + (t / LM) * PM + t % LM;
            double m[LM];
            rows_down<LX>(Jm, [&](int k) { return c[k * LX * PM]; }, m);
            SEM_GLOBAL double* out = gfieldw<double>(R, F_HRM) + (long long)e * LM * LM * LM + t;
#pragma unroll
            for (int k = 0; k < LM; ++k)
                if (live) out[LM * LM * k] = m[k];
        }
    }
    block_sync_lds();
    {   // y back
        double* x = sA + p * LX * P + q;
        double v[LX];
#pragma unroll
        for (int b = 0; b < LX; ++b) v[b] = x[b * P];
        rows_up<LX>(Sy, v, [&](int b, double s) { x[b * P] = s; });
    }
    block_sync_lds();
    {   // x back
        double* x = sA + t * P;
        double v[LX];
#pragma unroll
        for (int a = 0; a < LX; ++a) v[a] = x[a];
        rows_up<LX>(Sx, v, [&](int a, double s) { x[a] = s; });
    }
    block_sync_lds();
    SEM_GLOBAL double* u = gfieldw<double>(R, F_HSF) + base + t;
#pragma unroll
    for (int k = 0; k < LX; ++k)
        if (live) u[L2 * k] = sA[(k * LX + p) * P + q];
}

// ---------------------------------------------------------------- middle level, down
// hs_mepb(LM) elements per workgroup (one request per workgroup)
template <int LM>
__global__ void __launch_bounds__(hs_mepb(LM) * LM * LM) hs_mid_kernel(Batch bt, int lx, int gate)
{
    constexpr int L2 = LM * LM, L3 = L2 * LM, N = LM - 1, EP = hs_mepb(LM);
    __shared__ double sA[EP * L3], sB[EP * L3];
    __shared__ double sS[3 * L2], sLam[3 * LM], sJc[2 * LM], sC[EP * 2 * L2];
    const int g = blockIdx.x;
    const int ri = find_req(bt.hm, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    if (!gate_ok(R, gate)) return;
    const int t = threadIdx.x, el = t / L2, ij = t - el * L2, i = ij % LM, j = ij / LM;
    const int e = (g - bt.hm[ri]) * EP + el;
    const bool live = e < R->E;
    const int ee = live ? e : 0;        // lanes past the last element work on element 0 and store nothing
    const HsOff o = hs_off(lx, R->nel);
    const SEM_GLOBAL double* tb = gfield<double>(R, F_HST);
    for (int q = t; q < 3 * L2; q += EP * L2) sS[q] = tb[o.Sm + q];
    for (int q = t; q < 3 * LM; q += EP * L2) sLam[q] = tb[o.Lm + q];
    for (int q = t; q < 2 * LM; q += EP * L2) sJc[q] = tb[o.Jc + q];
    __syncthreads();
    int ex, ey, ez;
    elem_xyz(ee, R->nel, ex, ey, ez);
    const SEM_GLOBAL double* rm = gfield<double>(R, F_HRM);
    double v[LM];
    // the assembled middle residual: sum of the element contributions
    copies<LM>(rm, R->nel, ex, ey, ez, i, j, v);
    // coarse restriction of this element: c8 = Jc^T Jc^T Jc^T (r_m / mult)
    {
        double c0 = 0.0, c1 = 0.0;
#pragma unroll
        for (int k = 0; k < LM; ++k) {
            const double x = v[k] * inv_mult(i, j, k, N);
            c0 += sJc[k * 2 + 0] * x;
            c1 += sJc[k * 2 + 1] * x;
        }
        double* C = sC + el * 2 * L2;
        C[0 * L2 + j * LM + i] = c0;
        C[1 * L2 + j * LM + i] = c1;
        __syncthreads();
        if (ij < 8 && live) {
            const int ca = ij & 1, cb = (ij >> 1) & 1, cc = ij >> 2;
            double s = 0.0;
            for (int b = 0; b < LM; ++b)
                for (int a = 0; a < LM; ++a) s += sJc[a * 2 + ca] * sJc[b * 2 + cb] * C[cc * L2 + b * LM + a];
            gfieldw<double>(R, F_HC8)[(long long)e * 8 + ij] = s;
        }
    }
    fdm_solve<LM>(v, sS, sLam, sA + el * L3, sB + el * L3, i, j);
    if (live) {
        SEM_GLOBAL double* u = gfieldw<double>(R, F_HSM) + (long long)e * L3;
#pragma unroll
        for (int k = 0; k < LM; ++k) u[i + LM * (j + LM * k)] = v[k];
    }
}

// ---------------------------------------------------------------- coarse level
// unique corner node (cx, cy, cz): the sum of the contributions of its 8 elements
__device__ __forceinline__ double corner_sum(const SEM_GLOBAL double* c8, int nx, int ny, int nz, int cx, int cy, int cz)
{
    const int xl = cx == 0 ? nx - 1 : cx - 1, yl = cy == 0 ? ny - 1 : cy - 1, zl = cz == 0 ? nz - 1 : cz - 1;
    double v[8], s = 0.0;
#pragma unroll
    for (int h = 0; h < 8; ++h) {
        const int e = (h & 1 ? xl : cx) + nx * ((h & 2 ? yl : cy) + ny * (h & 4 ? zl : cz));
        v[h] = c8[(long long)e * 8 + h];
    }
#pragma unroll
    for (int h = 0; h < 8; ++h) s += v[h];
    return s;
}

// Coarse fast diagonalisation, x and y directions of HS_CW columns x of one
// z-plane per workgroup (grid.x = z, grid.z = columns): FWD: out = (S_y^T x
// S_x^T) of the gathered corner sums, else out = (S_y x S_x) in.  A plane alone
// (32 workgroups at 32^3) leaves the chip idle behind two serial sums with their
// matrices in memory: 8.5 us a launch at 20^3, now 7.0 with the gather (was a
// launch of 4.8) and 4.8 back.
#define HS_CW 8
template <bool FWD>
__global__ void __launch_bounds__(256) hs_cxy_kernel(Batch bt, int lx, int src, int dst, int gate)
{
    __shared__ double sP[HS_CPLANE], sY[HS_CPLANE], sX[HS_NELMAX * HS_CW], sQ[HS_NELMAX * HS_CW];
    const ReqDesc* R = bt.r[blockIdx.y];
    if (!gate_ok(R, gate)) return;
    const int nx = R->nel[0], ny = R->nel[1], nz = R->nel[2];
    const int cz = blockIdx.x, x0 = blockIdx.z * HS_CW;
    if (cz >= nz || x0 >= nx) return;
    const int nw = nx - x0 < HS_CW ? nx - x0 : HS_CW, np = nx * ny;
    const HsOff o = hs_off(lx, R->nel);
    const SEM_GLOBAL double* tb = gfield<double>(R, F_HST);
    const SEM_GLOBAL double* Sx = tb + o.Sc[0];
    const SEM_GLOBAL double* Sy = tb + o.Sc[1];
    const SEM_GLOBAL double* in = gfield<double>(R, src);
    for (int q = threadIdx.x; q < np; q += blockDim.x)
        sP[q] = FWD ? corner_sum(in, nx, ny, nz, q % nx, q / nx, cz) : in[(long long)cz * np + q];
    // sX[a][x], sY[b][y]: the entry that multiplies input a (b) of output x (y)
    for (int q = threadIdx.x; q < nx * nw; q += blockDim.x) {
        const int x = q % nw, a = q / nw;
        sX[q] = FWD ? Sx[a * nx + x0 + x] : Sx[(x0 + x) * nx + a];
    }
    for (int q = threadIdx.x; q < ny * ny; q += blockDim.x) {
        const int y = q % ny, b = q / ny;
        sY[q] = FWD ? Sy[q] : Sy[y * ny + b];
    }
    __syncthreads();
    for (int q = threadIdx.x; q < nw * ny; q += blockDim.x) {
        const int x = q % nw, y = q / nw;
        double s = 0.0;
#pragma unroll 4
        for (int a = 0; a < nx; ++a) s += sX[a * nw + x] * sP[y * nx + a];
        sQ[q] = s;
    }
    __syncthreads();
    SEM_GLOBAL double* out = gfieldw<double>(R, dst) + (long long)cz * np + x0;
    for (int q = threadIdx.x; q < nw * ny; q += blockDim.x) {
        const int x = q % nw, y = q / nw;
        double s = 0.0;
#pragma unroll 4
        for (int b = 0; b < ny; ++b) s += sY[b * ny + y] * sQ[b * nw + x];
        out[y * nx + x] = s;
    }
}

// coarse fast diagonalisation, z direction of HS_CW columns x of one y-row per
// workgroup (grid.x = y, grid.z = columns): S_z^T, division by the eigenvalue
// sums (the constant mode is dropped), S_z
__global__ void __launch_bounds__(256) hs_cz_kernel(Batch bt, int lx, int src, int dst, int gate)
{
    __shared__ double sZ[HS_NELMAX * (HS_NELMAX + 1)], sP[HS_NELMAX * HS_CW], sQ[HS_NELMAX * HS_CW];
    const ReqDesc* R = bt.r[blockIdx.y];
    if (!gate_ok(R, gate)) return;
    const int nx = R->nel[0], ny = R->nel[1], nz = R->nel[2];
    const int cy = blockIdx.x, x0 = blockIdx.z * HS_CW;
    if (cy >= ny || x0 >= nx) return;
    const int nw = nx - x0 < HS_CW ? nx - x0 : HS_CW, pz = nz | 1;
    const HsOff o = hs_off(lx, R->nel);
    const SEM_GLOBAL double* tb = gfield<double>(R, F_HST);
    const SEM_GLOBAL double* Sz = tb + o.Sc[2];
    const SEM_GLOBAL double* in = gfield<double>(R, src) + x0 + (long long)nx * cy;
    for (int q = threadIdx.x; q < nw * nz; q += blockDim.x) sP[q] = in[q % nw + (long long)nx * ny * (q / nw)];
    for (int q = threadIdx.x; q < nz * nz; q += blockDim.x) sZ[q / nz * pz + q % nz] = Sz[q];
    __syncthreads();
    const double ly = tb[o.Lc[1] + cy];
    for (int q = threadIdx.x; q < nw * nz; q += blockDim.x) {
        const int x = q % nw, z = q / nw;
        double s = 0.0;
#pragma unroll 4
        for (int c = 0; c < nz; ++c) s += sZ[c * pz + z] * sP[c * nw + x];
        if (x0 + x == R->hs_c0[0] && cy == R->hs_c0[1] && z == R->hs_c0[2]) s = 0.0;
        else s /= tb[o.Lc[0] + x0 + x] + ly + tb[o.Lc[2] + z];
        sQ[q] = s;
    }
    __syncthreads();
    SEM_GLOBAL double* out = gfieldw<double>(R, dst) + x0 + (long long)nx * cy;
    for (int q = threadIdx.x; q < nw * nz; q += blockDim.x) {
        const int x = q % nw, z = q / nw;
        double s = 0.0;
#pragma unroll 4
        for (int c = 0; c < nz; ++c) s += sZ[z * pz + c] * sQ[c * nw + x];
        out[x + (long long)nx * ny * z] = s;
    }
}

// The whole coarse solve of a small grid in one workgroup: the same sums, one
// launch for the gather's and three more.
#define HS_CSN 16       // points per direction
#define HS_CSM 1024     // points
__global__ void __launch_bounds__(1024) hs_csmall_kernel(Batch bt, int lx, int gate)
{
    constexpr int P = HS_CSN + 1;
    __shared__ double sA[HS_CSM], sB[HS_CSM], sS[3][HS_CSN * P], sL[3][HS_CSN];
    const ReqDesc* R = bt.r[blockIdx.x];
    if (!gate_ok(R, gate)) return;
    const int nx = R->nel[0], ny = R->nel[1], nz = R->nel[2], np = nx * ny, n = np * nz;
    const HsOff o = hs_off(lx, R->nel);
    const SEM_GLOBAL double* tb = gfield<double>(R, F_HST);
    const SEM_GLOBAL double* c8 = gfield<double>(R, F_HC8);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int m = R->nel[d];
        for (int q = threadIdx.x; q < m * m; q += blockDim.x) sS[d][q / m * P + q % m] = tb[o.Sc[d] + q];
        for (int q = threadIdx.x; q < m; q += blockDim.x) sL[d][q] = tb[o.Lc[d] + q];
    }
    for (int q = threadIdx.x; q < n; q += blockDim.x) sA[q] = corner_sum(c8, nx, ny, nz, q % nx, q / nx % ny, q / np);
    __syncthreads();
    // to[q] = sum_a S[a][x] from[..a..] (fwd) or S[x][a] (back) along direction d
    auto along = [&](int d, bool fwd, const double* from, auto put) {
        const int m = R->nel[d], st = d == 0 ? 1 : d == 1 ? nx : np;
        for (int q = threadIdx.x; q < n; q += blockDim.x) {
            const int x = q / st % m;
            const double* f = from + q - x * st;
            const double* S = sS[d] + (fwd ? x : x * P);
            const int ss = fwd ? P : 1;
            double s = 0.0;
#pragma unroll 4
            for (int a = 0; a < m; ++a) s += S[a * ss] * f[a * st];
            put(q, s);
        }
        __syncthreads();
    };
    auto toA = [&](int q, double s) { sA[q] = s; };
    auto toB = [&](int q, double s) { sB[q] = s; };
    along(0, true, sA, toB);
    along(1, true, sB, toA);
    along(2, true, sA, [&](int q, double s) {
        const int x = q % nx, y = q / nx % ny, z = q / np;
        if (x == R->hs_c0[0] && y == R->hs_c0[1] && z == R->hs_c0[2]) s = 0.0;
        else s /= sL[0][x] + sL[1][y] + sL[2][z];
        sB[q] = s;
    });
    along(2, false, sB, toA);
    along(0, false, sA, toB);
    SEM_GLOBAL double* out = gfieldw<double>(R, F_HCB);
    along(1, false, sB, [&](int q, double s) { out[q] = s; });
}

// ---------------------------------------------------------------- middle level, up
template <int LM>
__global__ void __launch_bounds__(hs_mepb(LM) * LM * LM) hs_midup_kernel(Batch bt, int lx, int gate)
{
    constexpr int L2 = LM * LM, L3 = L2 * LM, EP = hs_mepb(LM);
    __shared__ double sJc[2 * LM];
    __shared__ double sE[EP * 8];
    const int g = blockIdx.x;
    const int ri = find_req(bt.hm, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    if (!gate_ok(R, gate)) return;
    const int t = threadIdx.x, el = t / L2, ij = t - el * L2, i = ij % LM, j = ij / LM;
    const int e = (g - bt.hm[ri]) * EP + el;
    const bool live = e < R->E;
    const int ee = live ? e : 0;
    const HsOff o = hs_off(lx, R->nel);
    const SEM_GLOBAL double* tb = gfield<double>(R, F_HST);
    for (int q = t; q < 2 * LM; q += EP * L2) sJc[q] = tb[o.Jc + q];
    int ex, ey, ez;
    elem_xyz(ee, R->nel, ex, ey, ez);
    const int nx = R->nel[0], ny = R->nel[1], nz = R->nel[2];
    if (ij < 8) {
        const int a = ij & 1, b = (ij >> 1) & 1, c = ij >> 2;
        const int cx = (ex + a) % nx, cy = (ey + b) % ny, cz = (ez + c) % nz;
        sE[el * 8 + ij] = gfield<double>(R, F_HCB)[cx + nx * (cy + ny * cz)];
    }
    __syncthreads();
    if (!live) return;
    const double* E8 = sE + el * 8;
    double v[LM];
    const double rm = copies<LM>(gfield<double>(R, F_HSM), R->nel, ex, ey, ez, i, j, v);
    SEM_GLOBAL double* zm = gfieldw<double>(R, F_HZM) + (long long)e * L3;
#pragma unroll
    for (int k = 0; k < LM; ++k) {
        double p = 0.0;
        for (int c = 0; c < 2; ++c)
            for (int b = 0; b < 2; ++b)
                for (int a = 0; a < 2; ++a)
                    p += E8[a + 2 * (b + 2 * c)] * sJc[i * 2 + a] * sJc[j * 2 + b] * sJc[k * 2 + c];
        zm[i + LM * (j + LM * k)] = v[k] * (k == 0 || k == LM - 1 ? 0.5 * rm : rm) + p;   // the product is exact
    }
}

// ---------------------------------------------------------------- fine level, up
// z -> F_HZ (the operator's input) and Z_J of F_HZS (the cycle end's x update), type TZ
//
// Bound by memory and the latency of the copies; us a launch, lines and batched
// copies against one copy at a time: fp64 20^3, LX = 10 95 -> 68 (40 for the
// bytes), 32^3, LX = 8 169 -> 126, fp32 basis 92 -> 67; 12 of 4..9^3 17.4 -> 8.8.
template <int LX, typename TZ>
__global__ void __launch_bounds__(hs_fepb(LX) * LX * LX) hs_up_kernel(Batch bt, HsFine hf, int gate)
{
    constexpr int LM = hs_lxm(LX), LM2 = LM * LM, L2 = LX * LX, L3 = L2 * LX, N = LX - 1, P = LX | 1;
    constexpr int EP = hs_fepb(LX);
    __shared__ double sAs[EP * LM2 * P], sBs[EP * LM * L2];   // [c][b][i], [c][j][i]
    const int g = blockIdx.x;
    const int ri = find_req(hf.p, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    if (!gate_ok(R, gate)) return;
    const int el = EP > 1 ? threadIdx.x / L2 : 0, t = threadIdx.x - el * L2, i = t % LX, j = t / LX;
    const int e0 = (g - hf.p[ri]) * EP + el;
    const bool live = e0 < R->E;
    const int e = live ? e0 : 0;
    double* const sA = sAs + el * LM2 * P;
    double* const sB = sBs + el * LM * L2;
    const HsOff o = hs_off(LX, R->nel);
    Rows<LM, double> Jm;
    Jm.set((const double*)gfield<double>(R, F_HST) + o.J);
    int ex, ey, ez;
    elem_xyz(e, R->nel, ex, ey, ez);
    double v[LX];
    const double rm = copies<LX>(gfield<double>(R, F_HSF), R->nel, ex, ey, ez, i, j, v);
    // J3 z_m by lines: x (c, b), y (c, i), z (i, j)
    const SEM_GLOBAL double* zm = gfield<double>(R, F_HZM) + (long long)e * LM2 * LM;
    double x[LM];
    if (t < LM2) {
#pragma unroll
        for (int a = 0; a < LM; ++a) x[a] = zm[t * LM + a];
        rows_up<LX>(Jm, x, [&](int q, double p) { sA[t * P + q] = p; });
    }
    block_sync_lds();
    if (t < LM * LX) {
        const double* c = sA + (t / LX) * LM * P + t % LX;
#pragma unroll
        for (int b = 0; b < LM; ++b) x[b] = c[b * P];
        rows_up<LX>(Jm, x, [&](int q, double p) { sB[(t / LX) * L2 + q * LX + t % LX] = p; });
    }
    block_sync_lds();
#pragma unroll
    for (int c = 0; c < LM; ++c) x[c] = sB[c * L2 + t];
    const long long base = (long long)e * L3 + t;
    SEM_GLOBAL TZ* hz = gfieldw<TZ>(R, F_HZ) + base;
    SEM_GLOBAL TZ* zj = gfieldw<TZ>(R, F_HZS) + (long long)gp(R->I)[I_GJ] * R->np + base;
    rows_up<LX>(Jm, x, [&](int k, double p) {
        // (a product with a power of two is exact: fused or not, the same bits)
        const TZ z = (TZ)(v[k] * (k == 0 || k == N ? 0.5 * rm : rm) + p);
        if (live) {
            hz[L2 * k] = z;
            zj[L2 * k] = z;
        }
    });
}

template <int LX>
static void hsmg_go(const Batch& b, int tb, int gate, hipStream_t s)
{
    constexpr int LM = hs_lxm(LX);
    HsFine hf;
    hf.p[0] = 0;
    for (int i = 0; i < b.n; ++i) hf.p[i + 1] = hf.p[i] + (b.el[i + 1] - b.el[i] + hs_fepb(LX) - 1) / hs_fepb(LX);
    for (int i = b.n; i < SEM_MAXB; ++i) hf.p[i + 1] = hf.p[b.n];
    const int ne = hf.p[b.n], nt = hs_fepb(LX) * LX * LX;
    if (ne == 0) return;
    if (tb == P64) hipLaunchKernelGGL((hs_down_kernel<LX, double>), dim3(ne), dim3(nt), 0, s, b, hf, gate);
    else hipLaunchKernelGGL((hs_down_kernel<LX, float>), dim3(ne), dim3(nt), 0, s, b, hf, gate);
    constexpr int EP = hs_mepb(LM);
    const int nmb = b.hm[b.n];
    hipLaunchKernelGGL((hs_mid_kernel<LM>), dim3(nmb), dim3(EP * LM * LM), 0, s, b, LX, gate);
    // One workgroup while a thread has one point of the grid and the three
    // matrices fit beside it: 12 grids of 4..9^3 10.0 us against 17.5 in four
    // launches, 5 of 4..8^3 5.9 against 14.4.  At 20^3 (8000 points) the three
    // launches take 17.6 us and one workgroup would have eight rounds.
    if (b.cmax <= HS_CSN && b.ncmax <= HS_CSM) {
        hipLaunchKernelGGL(hs_csmall_kernel, dim3(b.n), dim3(1024), 0, s, b, LX, gate);
    } else {
        // F_HC8 -> (gather, x, y fwd) F_HCB -> (z) F_HCA -> (x, y back) F_HCB
        const dim3 cp(b.cmax, b.n, (b.cmax + HS_CW - 1) / HS_CW);
        hipLaunchKernelGGL((hs_cxy_kernel<true>), cp, dim3(256), 0, s, b, LX, (int)F_HC8, (int)F_HCB, gate);
        hipLaunchKernelGGL(hs_cz_kernel, cp, dim3(256), 0, s, b, LX, (int)F_HCB, (int)F_HCA, gate);
        hipLaunchKernelGGL((hs_cxy_kernel<false>), cp, dim3(256), 0, s, b, LX, (int)F_HCA, (int)F_HCB, gate);
    }
    hipLaunchKernelGGL((hs_midup_kernel<LM>), dim3(nmb), dim3(EP * LM * LM), 0, s, b, LX, gate);
    if (tb == P64) hipLaunchKernelGGL((hs_up_kernel<LX, double>), dim3(ne), dim3(nt), 0, s, b, hf, gate);
    else hipLaunchKernelGGL((hs_up_kernel<LX, float>), dim3(ne), dim3(nt), 0, s, b, hf, gate);
}

void launch_hsmg(const Batch& b, int lx, int tb, int gate, hipStream_t s)
{
    switch (lx) {
    case 5: hsmg_go<5>(b, tb, gate, s); break;
    case 6: hsmg_go<6>(b, tb, gate, s); break;
    case 7: hsmg_go<7>(b, tb, gate, s); break;
    case 8: hsmg_go<8>(b, tb, gate, s); break;
    case 9: hsmg_go<9>(b, tb, gate, s); break;
    case 10: hsmg_go<10>(b, tb, gate, s); break;
    case 11: hsmg_go<11>(b, tb, gate, s); break;
    case 12: hsmg_go<12>(b, tb, gate, s); break;
    default: break;
    }
}

}  // namespace semk
