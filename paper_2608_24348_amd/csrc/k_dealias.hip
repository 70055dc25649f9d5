// Dealiased convection: the convective term integrated on LXD = ceil(3 LX / 2)
// Gauss-Legendre points per direction (the 3/2 rule) instead of by
// collocation on the GLL points:
//   BN_f(l) = - sum_q W_q phi_l(z_q) sum_c u_c(z_q) sum_a (dr_a/dx_c)(z_q) (du_f/dr_a)(z_q)
// with W = jac * (Gauss-Legendre weights).  The metric terms W dr_a/dx_c at
// the fine points are computed once per mesh (dealias_geom_kernel) from the
// interpolated coordinates.  Per element (one workgroup), the velocity and
// its reference derivatives are taken to the fine points by staged
// one-dimensional contractions along whole lines; the contravariant velocity
// V_a = sum_c u_c W dr_a/dx_c stays in registers (each thread owns a fine
// line of the third index), and the weighted integrand goes back to the GLL
// points by the transposed contractions.
#include "k_lines.h"

#include <type_traits>

namespace semk {

template <int LX> struct Dl {
    static constexpr int LXD = (3 * LX + 1) / 2;
    static constexpr int N3 = LX * LX * LX;
    static constexpr int ND3 = LXD * LXD * LXD;
    static constexpr int NT = ND3 <= 1728 ? 256 : 512;
    static constexpr int NQ = (ND3 + NT - 1) / NT;
    static constexpr int NA = LXD * LX * LX;
    static constexpr int NB = LXD * LXD * LX;
};

// tables after the GLL tables: fp64 [D lx^2][w lx][xi lx][1/mult lx^3][I][ID][wz],
// fp32 [D lx^2][w lx][xi lx][I][ID][wz]; I, ID are LXD x LX, wz has LXD entries
template <int LX> __device__ __forceinline__ int dl_off64() { return LX * LX + 2 * LX + LX * LX * LX; }
template <int LX> __device__ __forceinline__ int dl_off32() { return LX * LX + 2 * LX; }

// out[(k LXD + j) LXD + i] = sum_{a,b,c} A1[i][a] A2[j][b] A3[k][c] in[(c LX + b) LX + a]
template <int LX, typename C>
__device__ __forceinline__ void interp3(const C* A1, const C* A2, const C* A3, const C* in, C* tA, C* tB, C* out)
{
    constexpr int LXD = Dl<LX>::LXD, NT = Dl<LX>::NT;
    const int t = threadIdx.x;
    for (int idx = t; idx < LX * LX * LXD; idx += NT) {
        const int i = idx % LXD, kj = idx / LXD;
        C s = 0;
#pragma unroll
        for (int a = 0; a < LX; ++a) s += A1[i * LX + a] * in[kj * LX + a];
        tA[idx] = s;
    }
    __syncthreads();
    for (int idx = t; idx < LX * LXD * LXD; idx += NT) {
        const int i = idx % LXD, r = idx / LXD, j = r % LXD, k = r / LXD;
        C s = 0;
#pragma unroll
        for (int b = 0; b < LX; ++b) s += A2[j * LX + b] * tA[(k * LX + b) * LXD + i];
        tB[idx] = s;
    }
    __syncthreads();
    for (int idx = t; idx < LXD * LXD * LXD; idx += NT) {
        const int i = idx % LXD, r = idx / LXD, j = r % LXD, k = r / LXD;
        C s = 0;
#pragma unroll
        for (int c = 0; c < LX; ++c) s += A3[k * LX + c] * tB[(c * LXD + j) * LXD + i];
        out[idx] = s;
    }
    __syncthreads();
}

// fine-grid metric terms MF[e][a*3+c][q] = W_q (dr_a/dx_c)(z_q), fp64, from
// the coordinates of the GLL nodes (the same mapping as the GLL geometry)
template <int LX>
__global__ void __launch_bounds__(Dl<LX>::NT) dealias_geom_kernel(Batch bt, MeshParams mp)
{
    constexpr int LXD = Dl<LX>::LXD, N3 = Dl<LX>::N3, ND3 = Dl<LX>::ND3, NT = Dl<LX>::NT, NQ = Dl<LX>::NQ;
    __shared__ double sI[LXD * LX], sID[LXD * LX], swz[LXD], sxi[LX];
    __shared__ double sx[3][N3];
    __shared__ double F[ND3];
    __shared__ double tA[Dl<LX>::NA], tB[Dl<LX>::NB];
    const int g = blockIdx.x;
    const int ri = find_req(bt.eb, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    const int blk = g - bt.eb[ri];
    const int t = threadIdx.x;
    const SEM_GLOBAL double* tab = gp(R->D64);
    for (int q = t; q < LXD * LX; q += NT) {
        sI[q] = tab[dl_off64<LX>() + q];
        sID[q] = tab[dl_off64<LX>() + LXD * LX + q];
    }
    for (int q = t; q < LXD; q += NT) swz[q] = tab[dl_off64<LX>() + 2 * LXD * LX + q];
    for (int q = t; q < LX; q += NT) sxi[q] = tab[LX * LX + LX + q];
    __syncthreads();
    SEM_GLOBAL double* MF = gfieldw<double>(R, F_MFD64);
    for (int el = 0; el < R->epb; ++el) {
        const int e = blk * R->epb + el;
        if (e >= R->E) break;
        for (int p = t; p < N3; p += NT) {
            const int i = p % LX, j = (p / LX) % LX, k = p / (LX * LX);
            double xo[3];
            node_xyz(mp, sxi, e, i, j, k, xo);
            sx[0][p] = xo[0]; sx[1][p] = xo[1]; sx[2][p] = xo[2];
        }
        __syncthreads();
        SEM_GLOBAL double* me = MF + (long long)e * 9 * ND3;
        // J[c][a] = dx_c/dr_a at the fine points, parked in slot a*3+c
        for (int c = 0; c < 3; ++c)
            for (int a = 0; a < 3; ++a) {
                interp3<LX, double>(a == 0 ? sID : sI, a == 1 ? sID : sI, a == 2 ? sID : sI, sx[c], tA, tB, F);
                for (int r = 0; r < NQ; ++r) {
                    const int q = t + r * NT;
                    if (q < ND3) me[(a * 3 + c) * ND3 + q] = F[q];
                }
            }
        for (int r = 0; r < NQ; ++r) {
            const int q = t + r * NT;
            if (q >= ND3) break;
            double J[3][3];
            for (int c = 0; c < 3; ++c)
                for (int a = 0; a < 3; ++a) J[c][a] = me[(a * 3 + c) * ND3 + q];
            const double det = J[0][0] * (J[1][1] * J[2][2] - J[1][2] * J[2][1])
                             - J[0][1] * (J[1][0] * J[2][2] - J[1][2] * J[2][0])
                             + J[0][2] * (J[1][0] * J[2][1] - J[1][1] * J[2][0]);
            double inv[3][3];
            inv[0][0] = (J[1][1] * J[2][2] - J[1][2] * J[2][1]) / det;
            inv[0][1] = (J[0][2] * J[2][1] - J[0][1] * J[2][2]) / det;
            inv[0][2] = (J[0][1] * J[1][2] - J[0][2] * J[1][1]) / det;
            inv[1][0] = (J[1][2] * J[2][0] - J[1][0] * J[2][2]) / det;
            inv[1][1] = (J[0][0] * J[2][2] - J[0][2] * J[2][0]) / det;
            inv[1][2] = (J[0][2] * J[1][0] - J[0][0] * J[1][2]) / det;
            inv[2][0] = (J[1][0] * J[2][1] - J[1][1] * J[2][0]) / det;
            inv[2][1] = (J[0][1] * J[2][0] - J[0][0] * J[2][1]) / det;
            inv[2][2] = (J[0][0] * J[1][1] - J[0][1] * J[1][0]) / det;
            const int i = q % LXD, j = (q / LXD) % LXD, k = q / (LXD * LXD);
            const double W = det * swz[i] * swz[j] * swz[k];
            for (int a = 0; a < 3; ++a)
                for (int c = 0; c < 3; ++c) me[(a * 3 + c) * ND3 + q] = W * inv[a][c];
        }
        __syncthreads();
    }
}

// fp32 and element-scaled 16-bit copies of the fine-grid metric terms, each
// rounded once from fp64 (power-of-two scales keep the 16-bit rounding single)
template <typename T16>
__global__ void __launch_bounds__(256) dealias_cast_kernel(Batch bt, int per_elem, int want32, int want16)
{
    __shared__ double red[4];
    const int g = blockIdx.x;
    const int ri = find_req(bt.eb, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    const int blk = g - bt.eb[ri];
    const SEM_GLOBAL double* src = gfield<double>(R, F_MFD64);
    for (int el = 0; el < R->epb; ++el) {
        const int e = blk * R->epb + el;
        if (e >= R->E) break;
        const SEM_GLOBAL double* me = src + (long long)e * per_elem;
        if (want32) {
            SEM_GLOBAL float* dst = gfieldw<float>(R, F_MFD32) + (long long)e * per_elem;
            for (int p = threadIdx.x; p < per_elem; p += blockDim.x) dst[p] = (float)me[p];
        }
        if (want16) {
            double mx = 0.0;
            for (int p = threadIdx.x; p < per_elem; p += blockDim.x) mx = fmax(mx, fabs(me[p]));
            mx = wave_max(mx);
            if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
            __syncthreads();
            mx = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
            __syncthreads();
            const double sc = mx > 0 ? exp2(ceil(log2(mx))) : 1.0;
            if (threadIdx.x == 0) gfieldw<float>(R, F_MFDSC)[e] = (float)sc;
            const int lx = R->lx;
            const int per16 = dl16_per_elem(lx);
            SEM_GLOBAL T16* dst = gfieldw<T16>(R, F_MFD16) + (long long)e * per16;
            if (dl16_lane(lx)) {
                // [tile][ac][g][m][r]: fine point (k' = 4g + r, n = 16 tile + m); zero outside
                const int nd = (3 * lx + 1) / 2, nn = nd * nd, ng = (nd + 3) / 4;
                for (int p = threadIdx.x; p < per16; p += blockDim.x) {
                    const int r = p & 3, m = (p >> 2) & 15, rest = p >> 6;
                    const int g = rest % ng, ac = (rest / ng) % 9, tile = rest / (ng * 9);
                    const int kk = 4 * g + r, n = 16 * tile + m;
                    const double v = (kk < nd && n < nn) ? me[(long long)ac * nd * nn + kk * nn + n] / sc : 0.0;
                    stg(dst + p, to<T16>(v));
                }
            } else {
                for (int p = threadIdx.x; p < per_elem; p += blockDim.x) stg(dst + p, to<T16>(me[p] / sc));
            }
        }
    }
}

template <typename TM> __device__ __forceinline__ int mfd_field() { return F_MFD16; }
template <> __device__ __forceinline__ int mfd_field<double>() { return F_MFD64; }
template <> __device__ __forceinline__ int mfd_field<float>() { return F_MFD32; }

// scale of an element's 16-bit terms
template <typename TM, typename C> __device__ __forceinline__ C mscale(const ReqDesc* R, int e)
{
    if constexpr (sizeof(TM) == 2) return (C)gfield<float>(R, F_MFDSC)[e];
    else return (C)1;
}

// ------------------------------------------------------------------
// BN = dealiased -B (u . grad) u.  A thread takes a whole line through a
// one-dimensional contraction, its inputs in registers and the matrix shared
// by the wave, so a line of LX values becomes LXD for LX + LXD LDS accesses.
// On the third index a thread owns the fine line (j', i') of the element: V_a,
// the integrand T and the transposed contraction back to LX values never leave
// its registers (15 LX LXD multiply-adds for 9 LX LDS reads).  Per element the
// I I u_c stay in LDS for all three components (the third-index derivative
// reads them again); the other two derivatives of a component pass through one
// buffer.
//   LDS: sIP [3][LX][NN], sB [LX][NN], sY [LX][LXD][LX|1] (then [NL][LXD|1]), for DPP I and ID
// Every sum runs over its index in ascending order from zero with fused
// multiply-adds; T adds its terms in the order K0, K1, K2.
//
// Bound by memory at LX <= 7 (the metric terms: 9 of 15 words at 3.4 times the
// points), above by waiting: in fp64 one workgroup of four (LX = 10) or six (12)
// waves a CU.  Counters there, LX = 10 and 12: VALU busy 24 and 32%, LDS 12 and 18%
// of the cycles (27 and 16% of that in conflicts), waves waiting 49 and 62% of
// theirs; 2.06 GB read from memory at LX = 12 where 1.89 are needed (977 us, 396 for
// the bytes).  A tile form on matrix cores pads lines of LX and LXD to 4 and 16, and
// passes V and T of a component through LDS; lines pad only the last of their waves.
// us a call, tile form (LX <= 10) or one thread a point (11, 12) before, lines now:
//   LX, elements     fp64          fp32          16-bit terms
//    3, 40^3         439 -> 245    358 -> 133    369 -> 147
//    4, 32^3         327 -> 162    245 -> 95     252 -> 106
//    5, 32^3         665 -> 303    363 -> 186    377 -> 145
//    6, 24^3         443 -> 222    251 -> 150    274 -> 133
//    7, 32 32 16     783 -> 459    390 -> 254    392 -> 234
//    8, 32^3        1718 -> 1656   829 -> 742    782 -> 722
//    9, 22^3        2396 -> 785    586 -> 415    535 -> 415
//   10, 20^3        2302 -> 1125   577 -> 443    515 -> 420
//   11, 18^3        3161 -> 1131  1954 -> 818   1960 -> 817
//   12, 16^3        2388 -> 977   1298 -> 697   1291 -> 678
// and with few elements, 2^3: LX = 3 45 -> 11, 8 48 -> 25, 12 275 -> 51 in fp64.
template <int LX, typename C> struct Dn {
    static constexpr int LXD = (3 * LX + 1) / 2, NL = LX * LX, NN = LXD * LXD, N3 = NL * LX, ND3 = NN * LXD;
    static constexpr int LJ = LX | 1, LP = LXD | 1;   // odd row strides: lanes a row apart fall in different banks
    static constexpr int cmax(int a, int b) { return a > b ? a : b; }
    static constexpr int YS = cmax(LX * LXD * LJ, NL * LP);
    static constexpr bool DPP = LX > 11;   // matrix entries by row broadcast (below)
    static constexpr int TOTAL = 4 * LX * NN + YS + (DPP ? 2 * LXD * LX : 0);
    static constexpr int NW = (NN + 63) / 64, NT = 64 * NW;
    static_assert(TOTAL * (int)sizeof(C) <= 160 * 1024, "LDS of a workgroup");
    // layers of metric terms in flight, the first of them (and u) loaded a stage
    // ahead.  With V and T of 18 rows in fp64 the registers do not hold that:
    // LX = 12, 1096 us with a ring of six and 977 with three on demand.
    static constexpr bool TIGHT = DPP && sizeof(C) == 8;
    static constexpr int RG = TIGHT ? 3 : LXD < 6 ? LXD : 6;
    // workgroups a CU by LDS, at most three, and the waves per SIMD that go with
    // them; more than two would spill V and T in fp64 (LX = 8: 2229 us at three,
    // 1625 at two) and at LX = 12
    static constexpr int WG = TOTAL * (int)sizeof(C) * 2 > 160 * 1024 ? 1 : TOTAL * (int)sizeof(C) * 3 > 160 * 1024 ? 2 : 3;
    static constexpr int WPE0 = (WG * NW + 3) / 4, WPE = (sizeof(C) == 8 || DPP) && WPE0 > 2 ? 2 : WPE0;
};

// The matrix entries of a line, two ways.
// By row broadcast: row o sits in one register, entry a in lane a of every
// 16-lane row of the wave (one LDS read for 3 rows), and a multiply-add takes it
// with the row broadcast of its DPP operand; fp64 runs at 0.9 of its plain rate
// so, fp32 at half.  By scalar registers (uniform loads): full rate, but a wave
// waits for each batch, and all that the waves of an element read (404 KB at
// LX = 12, fp64) comes through one scalar cache per two CUs.  us a call, fp64 /
// fp32 / 16-bit terms:
//          LX = 7         10               11               12
//   scalar  442/245/228   1118/432/412     1152/803/801     1273/945/901
//   DPP     472/279/284   1142/477/438     1231/899/895      967/670/650
// so the line lies between 11 and 12.  A DPP operand must not have been written
// by the two vector instructions before: the blocks begin with that wait,
// whatever the compiler puts ahead of them.  Lanes of the row must be on.
#define DL_OP64(d, c, x, n) "v_fmac_f64_dpp " d ", " c ", " x " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
#define DL_OP32(d, c, x, n) "v_fmac_f32_dpp " d ", " c ", " x " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
// three sums, one more input each: s_k += row_k[n] x
#define DL_UP(OP, x, n) OP("%0", "%3", x, n) OP("%1", "%4", x, n) OP("%2", "%5", x, n)
#define DL_UPS(OP, n0, n1, n2, n3, ...)                                                                                \
    if constexpr (N == 4)                                                                                              \
        asm("s_nop 1\n\t" DL_UP(OP, "%6", n0) DL_UP(OP, "%7", n1) DL_UP(OP, "%8", n2) DL_UP(OP, "%9", n3) __VA_ARGS__  \
            : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(x[0]), "v"(x[1]), "v"(x[2]), "v"(x[3])); \
    else if constexpr (N == 3)                                                                                         \
        asm("s_nop 1\n\t" DL_UP(OP, "%6", n0) DL_UP(OP, "%7", n1) DL_UP(OP, "%8", n2) __VA_ARGS__                      \
            : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(x[0]), "v"(x[1]), "v"(x[2])); \
    else if constexpr (N == 2)                                                                                         \
        asm("s_nop 1\n\t" DL_UP(OP, "%6", n0) DL_UP(OP, "%7", n1) __VA_ARGS__                                          \
            : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(x[0]), "v"(x[1]));            \
    else                                                                                                               \
        asm("s_nop 1\n\t" DL_UP(OP, "%6", n0) __VA_ARGS__                                                              \
            : "+v"(s[0]), "+v"(s[1]), "+v"(s[2]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(x[0]));
// s_k += sum over a = A .. A + N - 1 (ascending) of row_k[a] x[a - A], k = 0, 1, 2
template <int A, int N, typename C> __device__ __forceinline__ void up_block(C (&s)[3], const C (&c)[3], const C* x)
{
    if constexpr (sizeof(C) == 8) {
        if constexpr (A == 0) { DL_UPS(DL_OP64, 0, 1, 2, 3) }
        else if constexpr (A == 4) { DL_UPS(DL_OP64, 4, 5, 6, 7) }
        else { DL_UPS(DL_OP64, 8, 9, 10, 11) }
    } else {
        if constexpr (A == 0) { DL_UPS(DL_OP32, 0, 1, 2, 3) }
        else if constexpr (A == 4) { DL_UPS(DL_OP32, 4, 5, 6, 7) }
        else { DL_UPS(DL_OP32, 8, 9, 10, 11) }
    }
}
// one row into N sums: y[a] += row[a] v
#define DL_DN4(OP, c, v, n0, n1, n2, n3) OP("%0", c, v, n0) OP("%1", c, v, n1) OP("%2", c, v, n2) OP("%3", c, v, n3)
#define DL_DN3(OP, c, v, n0, n1, n2, n3) OP("%0", c, v, n0) OP("%1", c, v, n1) OP("%2", c, v, n2)
#define DL_DN2(OP, c, v, n0, n1, n2, n3) OP("%0", c, v, n0) OP("%1", c, v, n1)
#define DL_DN1(OP, c, v, n0, n1, n2, n3) OP("%0", c, v, n0)
#define DL_DNS(OP, n0, n1, n2, n3)                                                                                     \
    if constexpr (N == 4)                                                                                              \
        asm("s_nop 1\n\t" DL_DN4(OP, "%4", "%7", n0, n1, n2, n3) DL_DN4(OP, "%5", "%8", n0, n1, n2, n3)                \
                DL_DN4(OP, "%6", "%9", n0, n1, n2, n3)                                                                 \
            : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(v[0]), "v"(v[1]), "v"(v[2])); \
    else if constexpr (N == 3)                                                                                         \
        asm("s_nop 1\n\t" DL_DN3(OP, "%3", "%6", n0, n1, n2, n3) DL_DN3(OP, "%4", "%7", n0, n1, n2, n3)                \
                DL_DN3(OP, "%5", "%8", n0, n1, n2, n3)                                                                 \
            : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(v[0]), "v"(v[1]), "v"(v[2])); \
    else if constexpr (N == 2)                                                                                         \
        asm("s_nop 1\n\t" DL_DN2(OP, "%2", "%5", n0, n1, n2, n3) DL_DN2(OP, "%3", "%6", n0, n1, n2, n3)                \
                DL_DN2(OP, "%4", "%7", n0, n1, n2, n3)                                                                 \
            : "+v"(y[0]), "+v"(y[1]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(v[0]), "v"(v[1]), "v"(v[2]));             \
    else                                                                                                               \
        asm("s_nop 1\n\t" DL_DN1(OP, "%1", "%4", n0, n1, n2, n3) DL_DN1(OP, "%2", "%5", n0, n1, n2, n3)                \
                DL_DN1(OP, "%3", "%6", n0, n1, n2, n3)                                                                 \
            : "+v"(y[0]) : "v"(c[0]), "v"(c[1]), "v"(c[2]), "v"(v[0]), "v"(v[1]), "v"(v[2]));
// y[a - A] += row_0[a] v_0, then row_1[a] v_1, then row_2[a] v_2, a = A .. A + N - 1
template <int A, int N, typename C> __device__ __forceinline__ void down_block(C* y, const C (&c)[3], const C (&v)[3])
{
    if constexpr (sizeof(C) == 8) {
        if constexpr (A == 0) { DL_DNS(DL_OP64, 0, 1, 2, 3) }
        else if constexpr (A == 4) { DL_DNS(DL_OP64, 4, 5, 6, 7) }
        else { DL_DNS(DL_OP64, 8, 9, 10, 11) }
    } else {
        if constexpr (A == 0) { DL_DNS(DL_OP32, 0, 1, 2, 3) }
        else if constexpr (A == 4) { DL_DNS(DL_OP32, 4, 5, 6, 7) }
        else { DL_DNS(DL_OP32, 8, 9, 10, 11) }
    }
}
template <int LX, typename C, int A = 0> __device__ __forceinline__ void up_row(C (&s)[3], const C (&c)[3], const C (&x)[LX])
{
    if constexpr (A < LX) {
        up_block<A, (LX - A < 4 ? LX - A : 4), C>(s, c, x + A);
        up_row<LX, C, A + 4>(s, c, x);
    }
}
template <int LX, typename C, int A = 0> __device__ __forceinline__ void down_row(C (&y)[LX], const C (&c)[3], const C (&v)[3])
{
    if constexpr (A < LX) {
        down_block<A, (LX - A < 4 ? LX - A : 4), C>(y + A, c, v);
        down_row<LX, C, A + 4>(y, c, v);
    }
}

// a 1D matrix as line_up and line_down take it: by DPP this lane's entry of row 0 in LDS
template <typename C> struct LaneMat { const C* p; };
// (or RB rows at a time: more, up to the scalar registers, lose 2% at LX = 7, 8)
template <typename C> constexpr int dl_rb = sizeof(C) == 8 ? 3 : 6;
template <int LX, typename C, bool DPP> using Mat = std::conditional_t<DPP, LaneMat<C>, Rows<LX, C, dl_rb<C>>>;

// out(o, sum_a mat[o][a] x[a]) for the LXD rows o; every sum ascends in a from zero
template <int LX, int LXD, typename C, typename F>
__device__ __forceinline__ void line_up(Rows<LX, C, dl_rb<C>> mat, const C (&x)[LX], F out) { rows_up<LXD>(mat, x, out); }
template <int LX, int LXD, typename C, typename F>
__device__ __forceinline__ void line_up(LaneMat<C> mat, const C (&x)[LX], F out)
{
#pragma unroll
    for (int o = 0; o < LXD; o += 3) {
        C s[3], c[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s[k] = 0;
            c[k] = mat.p[(o + k < LXD ? o + k : o) * LX];
        }
        up_row<LX, C>(s, c, x);
        // (fp64: the next rows' entries stay unread till here, or V and T spill)
        if constexpr (sizeof(C) == 8) asm volatile("" : "+v"(s[0]), "+v"(s[1]), "+v"(s[2])::"memory");
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (o + k < LXD) out(o + k, s[k]);
    }
}
// y[a] = sum_o mat[o][a] in(o), ascending in o from zero
template <int LX, int LXD, typename C, typename F>
__device__ __forceinline__ void line_down(Rows<LX, C, dl_rb<C>> mat, F in, C (&y)[LX]) { rows_down<LXD>(mat, in, y); }
template <int LX, int LXD, typename C, typename F>
__device__ __forceinline__ void line_down(LaneMat<C> mat, F in, C (&y)[LX])
{
#pragma unroll
    for (int a = 0; a < LX; ++a) y[a] = 0;
#pragma unroll
    for (int o = 0; o < LXD; o += 3) {
        C c[3], v[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            c[k] = o + k < LXD ? mat.p[(o + k) * LX] : (C)0;   // past the last row nothing is added
            v[k] = o + k < LXD ? in(o + k) : (C)0;
        }
        down_row<LX, C>(y, c, v);
        if constexpr (sizeof(C) == 8) asm volatile("" : "+v"(y[0])::"memory");
    }
}

// K0, K1, K2: the order in which T adds V_r d_r u (0), V_s d_s u (1), V_t d_t u (2)
template <int LX, typename TM, typename C, int K0, int K1, int K2>
__global__ void __launch_bounds__((Dn<LX, C>::NT), (Dn<LX, C>::WPE)) conv_dealias_line_kernel(Batch bt, OpArrays io)
{
    using D = Dn<LX, C>;
    constexpr int LXD = D::LXD, NL = D::NL, NN = D::NN, N3 = D::N3, ND3 = D::ND3, LJ = D::LJ, LP = D::LP;
    __shared__ C lds[D::TOTAL];
    C* const sIP = lds;
    C* const sB = lds + 3 * LX * NN;
    C* const sY = sB + LX * NN;
    const int gb = blockIdx.x;
    const int ri = find_req(bt.el, bt.n, gb);
    const ReqDesc* R = bt.r[ri];
    if (!gate_ok(R, bt.gate)) return;
    const int e = gb - bt.el[ri];
    const int t = threadIdx.x;
    constexpr bool DPP = D::DPP;
    Mat<LX, C, DPP> mI, mD;
    if constexpr (DPP) {
        C* const sM = sY + D::YS;
        for (int q = t; q < 2 * LXD * LX; q += D::NT) {
            if constexpr (sizeof(C) == 8) sM[q] = gp(R->D64)[dl_off64<LX>() + q];
            else sM[q] = gp(R->D32)[dl_off32<LX>() + q];
        }
        mI.p = sM + ((t & 15) < LX ? t & 15 : LX - 1);
        mD.p = mI.p + LXD * LX;
        block_sync_lds();
    } else {
        const C* tab;
        if constexpr (sizeof(C) == 8) tab = R->D64 + dl_off64<LX>();
        else tab = R->D32 + dl_off32<LX>();
        mI.set(tab);
        mD.set(tab + LXD * LX);
    }

    // A wave whose first line is in range runs with every lane on, as the row
    // broadcasts need: lanes past the last line repeat it, and write what its
    // owner writes.
    const int t0 = __builtin_amdgcn_readfirstlane(t);
    auto lane_of = [&](int q0, int n) { return q0 + (t - t0) < n ? q0 + (t - t0) : n - 1; };
    const int tl = lane_of(t0, NL);

    // first index: sY[k][i'][j] = sum_a mat[i'][a] u_c[k][j][a], line t = (k, j)
    double xu[LX];
    auto load_u = [&](int c) {
        if (t0 < NL) {
            const SEM_GLOBAL double* u = op_in(R, io, F_U, c) + (long long)e * N3 + tl * LX;
#pragma unroll
            for (int a = 0; a < LX; ++a) xu[a] = u[a];
        }
    };
    auto first = [&](const Mat<LX, C, DPP>& mat, int c) {
        if (D::TIGHT) load_u(c);
        if (t0 < NL) {
            C x[LX];
#pragma unroll
            for (int a = 0; a < LX; ++a) x[a] = (C)xu[a];
            C* y = sY + (tl / LX) * LXD * LJ + tl % LX;
            line_up<LX, LXD>(mat, x, [&](int o, C v) { y[o * LJ] = v; });
        }
    };
    // second index: dst[k][j'][i'] = sum_b mat[j'][b] sY[k][i'][b], line q = (k, i')
    auto second = [&](const Mat<LX, C, DPP>& mat, C* dst) {
        for (int q0 = t0; q0 < LX * LXD; q0 += D::NT) {
            const int q = lane_of(q0, LX * LXD);
            const C* y = sY + q * LJ;
            C x[LX];
#pragma unroll
            for (int b = 0; b < LX; ++b) x[b] = y[b];
            C* o2 = dst + (q / LXD) * NN + q % LXD;
            line_up<LX, LXD>(mat, x, [&](int o, C v) { o2[o * LXD] = v; });
        }
    };
    const bool fine = t < NN;
    const int n = fine ? t : NN - 1;   // lanes past the plane repeat its last line and store nothing
    auto third_in = [&](const C* src, C (&x)[LX]) {
#pragma unroll
        for (int k = 0; k < LX; ++k) x[k] = src[k * NN + n];
    };

    // metric term (ac, k') of the line; 16-bit terms of lx <= 10 are lane-ordered
    const SEM_GLOBAL TM* me = gfield<TM>(R, mfd_field<TM>());
    constexpr bool LANE = sizeof(TM) == 2 && dl16_lane(LX);
    constexpr int NG = (LXD + 3) / 4;
    if constexpr (LANE) me += (long long)e * dl16_per_elem(LX) + (long long)(n >> 4) * 9 * NG * 64 + (n & 15) * 4;
    else me += (long long)e * 9 * ND3 + n;
    // row g = c LR + k' of the terms (a, c), a = 0..2: a ring of RG rows in flight,
    // loaded GR rows at a time (lane-ordered terms: four, in one load)
    constexpr int GR = LANE ? 4 : 1, LR = LANE ? 4 * NG : LXD;
    constexpr int RG = D::RG < GR ? GR : D::RG / GR * GR;
    TM mr[RG][3];
    auto load_m = [&](int g) {
        const int c = g / LR, k = g % LR;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const int ac = a * 3 + c;
            if constexpr (LANE) {
                typedef unsigned short U4 __attribute__((ext_vector_type(4)));
                const U4 q = *reinterpret_cast<const SEM_GLOBAL U4*>(me + (ac * NG + (k >> 2)) * 64);
#pragma unroll
                for (int j = 0; j < 4; ++j) mr[(g + j) % RG][a] = __builtin_bit_cast(TM, (unsigned short)q[j]);
            } else {
                mr[g % RG][a] = ldg(me + ac * ND3 + k * NN);
            }
        }
    };

    // ---- I I u_c of the three components, then V_a on the thread's fine line
    if constexpr (!D::TIGHT) load_u(0);
    auto start_m = [&]() {
#pragma unroll
        for (int g = 0; g < RG; g += GR) load_m(g);
    };
    if constexpr (!D::TIGHT) start_m();
    for (int c = 0; c < 3; ++c) {
        first(mI, c);
        if constexpr (!D::TIGHT) load_u(c < 2 ? c + 1 : 0);
        block_sync_lds();
        second(mI, sIP + c * LX * NN);
        block_sync_lds();
    }
    if constexpr (D::TIGHT) start_m();
    const C msc = mscale<TM, C>(R, e);
    C V[3][LXD];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        C x[LX];
        third_in(sIP + c * LX * NN, x);
        line_up<LX, LXD>(mI, x, [&](int k, C v) {
            const int g = c * LR + k;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                C mv = to<C>(mr[g % RG][a]);
                if constexpr (sizeof(TM) == 2) mv *= msc;
                V[a][k] = fma(v, mv, c == 0 ? (C)0 : V[a][k]);
            }
            // the row just read frees its slot
            if (k % GR == GR - 1 || k == LXD - 1) {
                const int g0 = g - k % GR;
                if (g0 + RG < 3 * LR) load_m(g0 + RG);
            }
        });
    }

    // ---- per component: T = sum_a V_a d_a u_f, back through the three indices
    for (int f = 0; f < 3; ++f) {
        C T[LXD];
#pragma unroll
        for (int k = 0; k < LXD; ++k) T[k] = 0;
        auto add = [&](auto kind_) {
            constexpr int kind = decltype(kind_)::value;
            const C* src = sIP + f * LX * NN;
            if constexpr (kind < 2) {
                first(kind == 0 ? mD : mI, f);
                block_sync_lds();
                second(kind == 0 ? mI : mD, sB);
                block_sync_lds();
                src = sB;
            }
            C x[LX];
            third_in(src, x);
            line_up<LX, LXD>(kind == 2 ? mD : mI, x, [&](int k, C v) { T[k] = fma(V[kind][k], v, T[k]); });
            // (the next write to sB or sIP comes after another barrier: every
            // kind that uses sB passes the one behind its first index)
        };
        add(std::integral_constant<int, K0>());
        add(std::integral_constant<int, K1>());
        add(std::integral_constant<int, K2>());
        if (!D::TIGHT && f < 2) load_u(f + 1);
        C z[LX];
        line_down<LX, LXD>(mI, [&](int k) { return T[k]; }, z);
        block_sync_lds();   // sB has been read
        if (fine) {
#pragma unroll
            for (int c = 0; c < LX; ++c) sB[c * NN + n] = z[c];
        }
        block_sync_lds();
        // transposed second index: sY[(c, b)][i'] = sum_j' I[j'][b] sB[c][j'][i'], line (c, i')
        for (int q0 = t0; q0 < LX * LXD; q0 += D::NT) {
            const int q = lane_of(q0, LX * LXD);
            const C* src = sB + (q / LXD) * NN + q % LXD;
            C y[LX];
            line_down<LX, LXD>(mI, [&](int o) { return src[o * LXD]; }, y);
            C* dst = sY + (q / LXD) * LX * LP + q % LXD;
#pragma unroll
            for (int b = 0; b < LX; ++b) dst[b * LP] = y[b];
        }
        block_sync_lds();
        // transposed first index: BN_f[c][b][a] = -sum_i' I[i'][a] sY[(c, b)][i'], line t = (c, b)
        if (t0 < NL) {
            const C* src = sY + tl * LP;
            C y[LX];
            line_down<LX, LXD>(mI, [&](int o) { return src[o]; }, y);
            SEM_GLOBAL double* o = op_out(R, io, F_BN, f) + (long long)e * N3 + t * LX;
            if (t < NL) {
#pragma unroll
                for (int a = 0; a < LX; ++a) o[a] = -(double)y[a];
            }
        }
        block_sync_lds();   // sY has been read
    }
}

#define DL_LX_SWITCH(lx, CALL) \
    switch (lx) { \
    case 3: CALL(3); break; case 4: CALL(4); break; case 5: CALL(5); break; case 6: CALL(6); break; \
    case 7: CALL(7); break; case 8: CALL(8); break; case 9: CALL(9); break; case 10: CALL(10); break; \
    case 11: CALL(11); break; case 12: CALL(12); break; default: break; }

void launch_dealias_geom(const Batch& b, int lx, const MeshParams& mp, int want32, int want16, hipStream_t s)
{
    if (b.eb[b.n] == 0) return;
#define GO(L) hipLaunchKernelGGL(dealias_geom_kernel<L>, dim3(b.eb[b.n]), dim3(Dl<L>::NT), 0, s, b, mp)
    DL_LX_SWITCH(lx, GO)
#undef GO
    if (want32 || want16) {
        const int nd = (3 * lx + 1) / 2;
        const int per = 9 * nd * nd * nd;
        if (want16 == PBF)
            hipLaunchKernelGGL(dealias_cast_kernel<__hip_bfloat16>, dim3(b.eb[b.n]), dim3(256), 0, s, b, per, want32, 1);
        else
            hipLaunchKernelGGL(dealias_cast_kernel<__half>, dim3(b.eb[b.n]), dim3(256), 0, s, b, per, want32,
                               want16 == P16 ? 1 : 0);
    }
}

// metric storage tm and arithmetic tc (tables in the arithmetic precision):
// (fp64, fp64), (fp32, fp64), (fp32, fp32) or (fp16/bf16, fp32)
void launch_conv_dealias(const Batch& b, int lx, int tm, int tc, hipStream_t s, const OpArrays* arrays)
{
    const OpArrays io = arrays ? *arrays : OpArrays{};
    if (b.eb[b.n] == 0) return;
    // the order of T's three terms: a step's fields answer to its last bit, so
    // each order and precision adds them as it always has
#define GO3(L, TM, C)                                                                                                  \
    do {                                                                                                               \
        constexpr bool swap = L <= 8 || (L <= 10 && sizeof(C) == 4), back = !swap && L <= 10;                          \
        hipLaunchKernelGGL((conv_dealias_line_kernel<L, TM, C, (swap ? 1 : back ? 2 : 0), (swap ? 0 : 1),              \
                                                     (swap || !back ? 2 : 0)>),                                        \
                           dim3(b.el[b.n]), dim3((Dn<L, C>::NT)), 0, s, b, io);                                        \
    } while (0)
    if (tm == P64) {
#define GO(L) GO3(L, double, double)
        DL_LX_SWITCH(lx, GO)
#undef GO
    } else if (tm == P16) {
#define GO(L) GO3(L, __half, float)
        DL_LX_SWITCH(lx, GO)
#undef GO
    } else if (tm == PBF) {
#define GO(L) GO3(L, __hip_bfloat16, float)
        DL_LX_SWITCH(lx, GO)
#undef GO
    } else if (tc == P64) {
#define GO(L) GO3(L, float, double)
        DL_LX_SWITCH(lx, GO)
#undef GO
    } else {
#define GO(L) GO3(L, float, float)
        DL_LX_SWITCH(lx, GO)
#undef GO
    }
#undef GO3
}

}  // namespace semk
