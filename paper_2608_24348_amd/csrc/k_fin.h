// Finalisation of Krylov reductions and the scalar logic of PCG, GMRES and
// the BDF/EXT step, run by a one-workgroup-per-request kernel after the
// producer of the partials.  Partials of a slot are added in a fixed order
// (fp64), so a request's scalars do not depend on its batch.  (Letting the
// last workgroup of the producer finalise instead needs a device-scope
// release per workgroup, an L2 write-back on this chip that costs far more
// than the separate launch.)
#pragma once
#include "k_common.h"

namespace semk {

// ------------------------------------------------------------------ finalise kernels
// fixed-order sums of the partials of NS slots (valid in thread 0): for each
// slot, thread t < 256 adds partials t, t+256, t+512, ... in that order, then the
// per-thread sums are added in a fixed tree.  The slots are read together,
// eight loads of each in flight, so a finaliser waits for one round of loads
// where it waited for NS.  red must hold 4 * NS values.
template <int NS>
static __device__ void slot_sums(const ReqDesc* R, const int (&slot)[NS], double (&out)[NS], double* red)
{
    constexpr int U = 8, bd = 256;
    const int t = threadIdx.x;
    double s[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) s[k] = 0.0;
    if (t < bd) {
        const SEM_GLOBAL double* p[NS];
        int cnt[NS], most = 0;
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            p[k] = gp(R->part) + (long long)slot[k] * R->pstride;
            cnt[k] = gp(R->I)[I_PCNT + slot[k]];
            most = max(most, cnt[k]);
        }
        for (int q = t; q < most; q += U * bd) {
            double a[NS][U];
#pragma unroll
            for (int k = 0; k < NS; ++k)
#pragma unroll
                for (int u = 0; u < U; ++u) a[k][u] = q + u * bd < cnt[k] ? p[k][q + u * bd] : 0.0;
#pragma unroll
            for (int k = 0; k < NS; ++k)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (q + u * bd < cnt[k]) s[k] += a[k][u];
        }
    }
#pragma unroll
    for (int k = 0; k < NS; ++k) s[k] = wave_sum(s[k]);
    __syncthreads();
    if (t < bd && (t & 63) == 0) {
#pragma unroll
        for (int k = 0; k < NS; ++k) red[(t >> 6) * NS + k] = s[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NS; ++k) {
        double v = 0.0;   // (defined in every thread: a caller returns it)
        if (t == 0)
            for (int w = 0; w < bd / 64; ++w) v += red[w * NS + k];
        out[k] = v;
    }
    __syncthreads();
}
static __device__ double slot_sum(const ReqDesc* R, int slot, double* red)
{
    const int sl[1] = {slot};
    double v[1];
    slot_sums<1>(R, sl, v, red);
    return v[0];
}
static __device__ double slot_max(const ReqDesc* R, int slot, double* red)
{
    double s = 0.0;
    const SEM_GLOBAL double* p = gp(R->part) + (long long)slot * R->pstride;
    const int cnt = gp(R->I)[I_PCNT + slot];
    for (int q = threadIdx.x; q < cnt; q += blockDim.x) s = fmax(s, p[q]);
    s = wave_max(s);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    double m = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) m = fmax(m, red[w]);
    __syncthreads();
    return m;
}

// fixed-order sums of nslots (<= 32) consecutive slots at once: partials g,
// g+8, g+16, ... of a slot are added in that order for g = 0..7, then the 8
// group sums in group order.  A wave to a slot: it reads 256 partials coalesced
// into LDS (the next 256 in flight meanwhile) and its lanes 0..7 walk the eight
// chains there.  With a slot to a thread, eight scattered loads in flight, the
// 1142 partials of a 20^3, N = 9 Arnoldi step took 12 us.  stage must hold 256
// values per wave, out nslots.
static __device__ void multi_slot_sum(const ReqDesc* R, int slot0, int nslots, double* out, double* stage)
{
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    double* st = stage + (threadIdx.x >> 6) * 256;
    for (int k = threadIdx.x >> 6; k < nslots; k += nw) {
        const SEM_GLOBAL double* p = gp(R->part) + (long long)(slot0 + k) * R->pstride;
        const int cnt = gp(R->I)[I_PCNT + slot0 + k];
        double a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = lane + 64 * u < cnt ? p[lane + 64 * u] : 0.0;
        double acc = 0.0;
        for (int q0 = 0; q0 < cnt; q0 += 256) {
#pragma unroll
            for (int u = 0; u < 4; ++u) st[lane + 64 * u] = a[u];
            const int q1 = q0 + 256 + lane;
#pragma unroll
            for (int u = 0; u < 4; ++u) a[u] = q1 + 64 * u < cnt ? p[q1 + 64 * u] : 0.0;
            lds_handoff<true>();
            if (lane < 8) {
                const int n = min(256, cnt - q0);
                int q = lane;
                for (; q + 56 < n; q += 64) {
                    double b[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) b[u] = st[q + 8 * u];
#pragma unroll
                    for (int u = 0; u < 8; ++u) acc += b[u];
                }
                for (; q < n; q += 8) acc += st[q];
            }
            lds_handoff<true>();
        }
        if (lane < 8) st[lane] = acc;
        lds_handoff<true>();
        if (lane == 0) {
            double v = 0.0;
            for (int g = 0; g < 8; ++g) v += st[g];
            out[k] = v;
        }
        lds_handoff<true>();
    }
    __syncthreads();
}

static __device__ __forceinline__ bool finite(double v) { return isfinite(v); }

// The scalar logic of one request, run by one workgroup of SEM_FIN_THREADS (red
// holds up to six slots of four waves).  Vectors of the small GMRES
// system are read by all threads at once into LDS: a thread that walks them in
// global memory waits about 1 us for each dependent element.  ri is the
// request's position in its batch (host arrays).
static __device__ __noinline__ void fin_body(ReqDesc* R, int ri, const FinArgs a)
{
    __shared__ double red[32];
    __shared__ double sums[SEM_MAXM + 2];
    __shared__ double stage[SEM_FIN_THREADS / 64 * 256];  // the partial sums' staging, or the small GMRES system
    __shared__ double shc[SEM_MAXM + 1], shs[SEM_MAXM + 1];
    __shared__ int jsolve;
    SEM_GLOBAL double* S = gp(R->S);
    SEM_GLOBAL int* I = gp(R->I);
    const int t = threadIdx.x;
    if (a.gate2 >= 0 && !I[a.gate2]) return;  // uniform per workgroup
    switch (a.op) {
    case FIN_VINIT: {
        const int sl[3] = {R_A, R_A + 1, R_A + 2};
        double v[3];
        slot_sums<3>(R, sl, v, red);
        for (int c = 0; c < 3; ++c) {
            const double s = v[c];
            if (t == 0) {
                double rn = sqrt(s);
                S[S_R0 + c] = rn;
                S[S_RN + c] = rn;
                bool act = rn > S[S_VTOL] && I[I_VREF + c] < I[I_VMAXREF];
                if (!finite(rn)) { I[I_NAN] = 1; act = false; }
                if (act) I[I_VREF + c] += 1;
                I[I_VACT + c] = act ? 1 : 0;
            }
        }
        break;
    }
    case FIN_PCG_RHO: {
        const int sl[3] = {R_B, R_B + 1, R_B + 2};
        double v[3];
        slot_sums<3>(R, sl, v, red);
        for (int c = 0; c < 3; ++c)
            if (t == 0 && I[I_VACT + c]) S[S_RHO + c] = v[c];
        break;
    }
    case FIN_PCG_ALPHA: {
        // (an idle component's slot is summed too; its result is not used)
        const int sl[3] = {R_A, R_A + 1, R_A + 2};
        double v[3];
        slot_sums<3>(R, sl, v, red);
        for (int c = 0; c < 3; ++c)
            if (t == 0 && I[I_VACT + c]) S[S_ALPHA + c] = S[S_RHO + c] / v[c];
        break;
    }
    case FIN_PCG_BETA: {
        const int sl[6] = {R_B, R_C, R_B + 1, R_C + 1, R_B + 2, R_C + 2};
        double v[6];
        slot_sums<6>(R, sl, v, red);
        for (int c = 0; c < 3; ++c) {
            if (!I[I_VACT + c]) continue;
            const double rr = v[2 * c], rz = v[2 * c + 1];
            if (t == 0) {
                double rn = sqrt(rr);
                S[S_RN + c] = rn;
                I[I_VIT + c] += 1;
                if (!finite(rn)) { I[I_NAN] = 1; I[I_VACT + c] = 0; }
                else if (rn <= S[S_VTOL] || I[I_VIT + c] >= I[I_VMAXIT]) I[I_VACT + c] = 0;
                else { S[S_BETA + c] = rz / S[S_RHO + c]; S[S_RHO + c] = rz; }
            }
        }
        break;
    }
    case FIN_MEAN_UNIQUE: {
        double s = slot_sum(R, R_X3, red);
        if (t == 0) S[S_MEAN] = s / (double)R->nglob;
        break;
    }
    case FIN_MEAN_MASS: {
        double s = slot_sum(R, R_X3, red);
        if (t == 0) S[S_MEAN] = s / S[S_VOL];
        break;
    }
    case FIN_GM_H1:
    case FIN_GM_H2: {
        if (!I[I_GARN]) break;
        const int J = I[I_GJ];
        multi_slot_sum(R, R_GM, J + 1, sums, stage);
        // dots with the stored vectors, scaled to the normalised basis
        if (t <= J) S[(a.op == FIN_GM_H1 ? S_GHC : S_GH2) + t] = sums[t] * S[S_GVS + t];
        if (a.op == FIN_GM_H1) {
            double s = slot_sum(R, R_GMEAN, red);
            if (t == 0) S[S_GMEAN] = s / (double)R->nglob;
        }
        if (t == 0) I[I_GNORM] = 0;
        break;
    }
    case FIN_GM_COL: {
        if (!I[I_GARN]) break;
        const int m = I[I_GM];
        const int J = I[I_GJ];
        SEM_GLOBAL double* H = S + S_GH;
        if (t <= J) sums[t] = S[S_GHC + t] + S[S_GH2 + t];
        if (t < J) { shc[t] = S[S_GCS + t]; shs[t] = S[S_GSN + t]; }
        if (t == 0) jsolve = 0;
        double hn2 = slot_sum(R, R_GN, red);  // its barriers order the LDS reads below
        if (t == 0) {
            SEM_GLOBAL double* gg = S + S_GG;
            const double hn = sqrt(hn2);
            double x = sums[0];
            for (int i = 0; i < J; ++i) {
                const double y = sums[i + 1], c = shc[i], s = shs[i];
                sums[i] = fma(c, x, s * y);
                x = fma(c, y, -(s * x));
            }
            const double den = sqrt(fma(x, x, hn * hn));
            const double cj = x / den, sj = hn / den, gj = gg[J];
            sums[J] = den;
            H[(J + 1) * m + J] = 0.0;
            S[S_GCS + J] = cj;
            S[S_GSN + J] = sj;
            const double gn = -sj * gj;
            gg[J + 1] = gn;
            gg[J] = cj * gj;
            I[I_GIT] += 1;
            const bool bad = !finite(gn) || !finite(den);
            if (bad) I[I_NAN] = 1;
            if (bad || fabs(gn) <= S[S_PTOL] || hn == 0.0 || J + 1 == m || I[I_GIT] >= I[I_GMAXIT]) {
                const int jend = bad ? 0 : J + 1;
                jsolve = jend;
                I[I_GJEND] = jend;
                I[I_GARN] = 0;
                I[I_GEND] = 1;
                I[I_GENDAX] = 1;
                I[I_GNORM] = 0;
            } else {
                I[I_GJ] = J + 1;
                S[S_GVS + J + 1] = 1.0 / hn;
                I[I_GNORM] = 1;
            }
        }
        __syncthreads();
        if (t <= J) H[t * m + J] = sums[t];
        const int n = jsolve;  // uniform
        if (n > 0) {
            // y from the upper triangular system (column J is still in LDS)
            double* sH = stage;
            for (int q = t; q < n * n; q += blockDim.x) {
                const int r = q / n, c = q - r * n;
                sH[r * SEM_MAXM + c] = c == J ? sums[r] : r <= c ? H[r * m + c] : 0.0;
            }
            if (t < n) shc[t] = S[S_GG + t];
            __syncthreads();
            if (t == 0) {
                for (int r = n - 1; r >= 0; --r) {
                    double s = shc[r];
                    for (int k = r + 1; k < n; ++k) s -= sH[r * SEM_MAXM + k] * shs[k];
                    shs[r] = s / sH[r * SEM_MAXM + r];
                    S[S_GY + r] = shs[r];
                }
            }
        }
        break;
    }
    case FIN_GM_RESTART: {
        if (!I[I_GEND]) break;
        double s = slot_sum(R, R_GN, red);
        if (t == 0) {
            const double beta = sqrt(s);
            S[S_GBETA] = beta;
            I[I_GEND] = 0;
            I[I_GENDAX] = 0;
            if (!finite(beta)) I[I_NAN] = 1;
            if (!finite(beta) || beta <= S[S_PTOL] || I[I_GIT] >= I[I_GMAXIT]) {
                I[I_GACT] = 0; I[I_GARN] = 0; I[I_GNORM] = 0;
            } else {
                I[I_GJ] = 0;
                SEM_GLOBAL double* gg = S + S_GG;
                gg[0] = beta;  // (gg[j + 1] is written with column j, before it is read)
                S[S_GVS] = 1.0 / beta;
                I[I_GARN] = 1; I[I_GNORM] = 1;
            }
        }
        break;
    }
    case FIN_GM_START: {
        // fresh solve: the first cycle end computes r = b, or r = b - A x0
        // when the iterate starts from a nonzero projected guess
        if (t == 0) {
            const int x0 = R->proj_L > 0 && I[I_PRL] > 0;
            I[I_GJ] = 0; I[I_GJEND] = 0; I[I_GIT] = 0;
            I[I_GACT] = 1; I[I_GARN] = 0; I[I_GEND] = 1; I[I_GENDAX] = x0; I[I_GNORM] = 0;
        }
        break;
    }
    case FIN_PR_ALPHA: {
        const int l = I[I_PRL];
        multi_slot_sum(R, R_GM, l, sums, stage);
        if (t < l) S[S_PRA + t] = sums[t] * S[S_PRS + t];
        break;
    }
    case FIN_PR_POST: {
        if (t == 0) {
            const int full = I[I_PRL] >= R->proj_L;
            if (full) I[I_PRL] = 0;
            I[I_PRFULL] = full;
        }
        break;
    }
    case FIN_PR_BETA: {
        const int l = I[I_PRL];
        multi_slot_sum(R, R_GM, l + 1, sums, stage);
        if (t < l) {
            const double bi = sums[t] * S[S_PRS + t];
            S[S_PRB + t] = bi;
            shc[t] = bi;
        }
        __syncthreads();
        if (t == 0) {
            const double n2b = sums[l];
            double n2 = n2b;
            for (int i = 0; i < l; ++i) n2 -= shc[i] * shc[i];
            // a vector whose A-norm mostly lies in the space is dependent: dropped
            const int add = finite(n2b) && n2b > 0.0 && n2 > 1e-12 * n2b;
            I[I_PRADD] = add;
            if (add) S[S_PRS + l] = 1.0 / sqrt(n2);
        }
        break;
    }
    case FIN_PR_COMMIT: {
        if (t == 0 && I[I_PRADD]) I[I_PRL] += 1;
        break;
    }
    case FIN_COMMIT_CHECK: {
        // a captured step runs a fixed number of iterations: its correction,
        // lag rotation and projection update run only where every solve
        // stopped by itself within them (converged, hit its limit or met a
        // non-finite value); elsewhere the host re-runs the step
        if (t == 0) {
            const int done = !(I[I_VACT] | I[I_VACT + 1] | I[I_VACT + 2] | I[I_GACT]);
            I[I_COMMIT] = I[I_COMMIT + 1] = I[I_COMMIT + 2] = done;
            if (!done) I[I_PRADD] = 0;
        }
        break;
    }
    case FIN_DIAG: {
        const int sl[2] = {R_X0, R_X1};
        double v[2];
        slot_sums<2>(R, sl, v, red);
        const double ke = v[0], en = v[1];
        double md = slot_max(R, R_X2, red);
        double cr = slot_max(R, R_X4, red);
        if (t == 0) {
            S[S_KE] = ke / S[S_VOL];
            S[S_ENST] = en / S[S_VOL];
            S[S_MAXDIV] = md;
            S[S_CFLR] = cr;
            if (!finite(ke) || !finite(en)) I[I_NAN] = 1;
        }
        break;
    }
    case FIN_STEP_BEGIN: {
        if (t == 0) {
            const int torder = I[I_TORDER];
            const int k = I[I_STEP] + 1 < torder ? I[I_STEP] + 1 : torder;
            I[I_ORDER] = k;
            double b0, b1 = 0, b2 = 0, b3 = 0, a1 = 0, a2 = 0, a3 = 0;
            const double rate = S[S_CFLR];
            if (S[S_CFLT] > 0.0) {
                // adaptive step toward the target CFL, at most the configured dt,
                // and after the first step within [0.5, 1.1] of the previous one
                double dt = rate > 0.0 ? S[S_CFLT] / rate : S[S_DTMAX];
                if (I[I_STEP] > 0) {
                    const double prev = S[S_DTH];
                    if (dt > 1.1 * prev) dt = 1.1 * prev;
                    if (dt < 0.5 * prev) dt = 0.5 * prev;
                }
                if (dt > S[S_DTMAX]) dt = S[S_DTMAX];
                S[S_DTH + 2] = S[S_DTH + 1];
                S[S_DTH + 1] = S[S_DTH];
                S[S_DTH] = dt;
                S[S_DT] = dt;
                // BDF-k: derivative at t_{n+1} of the interpolant through the
                // last k+1 time levels; EXT-k: its value from the last k levels
                // (nodes measured back from t_{n+1}: 0, -h0, -h0-h1, -h0-h1-h2)
                double z[4];
                z[0] = 0.0;
                for (int q = 1; q < 4; ++q) z[q] = z[q - 1] - S[S_DTH + q - 1];
                double bb[4] = {0, 0, 0, 0}, aa[4] = {0, 0, 0, 0};
                double s0 = 0.0;
                for (int q = 1; q <= k; ++q) s0 += 1.0 / (z[0] - z[q]);
                bb[0] = dt * s0;
                for (int j = 1; j <= k; ++j) {
                    double nu_ = 1.0, de = 1.0, w = 1.0;
                    for (int q = 0; q <= k; ++q) {
                        if (q == j) continue;
                        de *= z[j] - z[q];
                        if (q != 0) {
                            nu_ *= z[0] - z[q];
                            w *= (z[0] - z[q]) / (z[j] - z[q]);
                        }
                    }
                    bb[j] = -dt * nu_ / de;
                    aa[j] = w;
                }
                b0 = bb[0]; b1 = bb[1]; b2 = bb[2]; b3 = bb[3];
                a1 = aa[1]; a2 = aa[2]; a3 = aa[3];
            } else if (k == 1) { b0 = 1.0; b1 = 1.0; a1 = 1.0; }
            else if (k == 2) { b0 = 1.5; b1 = 2.0; b2 = -0.5; a1 = 2.0; a2 = -1.0; }
            else { b0 = 11.0 / 6.0; b1 = 3.0; b2 = -1.5; b3 = 1.0 / 3.0; a1 = 3.0; a2 = -3.0; a3 = 1.0; }
            S[S_CFL] = S[S_DT] * rate;
            S[S_BETA0] = b0;
            S[S_BDF] = b1; S[S_BDF + 1] = b2; S[S_BDF + 2] = b3;
            S[S_EXT] = a1; S[S_EXT + 1] = a2; S[S_EXT + 2] = a3;
            S[S_H1] = S[S_NU];
            S[S_H2] = b0 / S[S_DT];
            const bool stale = I[I_STEP] == 0 || S[S_IDV_H1] != S[S_H1] || S[S_IDV_H2] != S[S_H2];
            I[I_IDVSTALE] = stale ? 1 : 0;
            S[S_IDV_H1] = S[S_H1];
            S[S_IDV_H2] = S[S_H2];
            S[S_MEAN + 0] = 0.0;
            for (int c = 0; c < 3; ++c) { I[I_VIT + c] = 0; I[I_VREF + c] = 0; I[I_VACT + c] = 0; }
        }
        break;
    }
    case FIN_STEP_END: {
        if (t == 0) {
            for (int c = 0; c < 3; ++c) {
                void* un = R->f[F_UL2 + c];          // holds u^{n+1}
                R->f[F_UL2 + c] = R->f[F_UL1 + c];
                R->f[F_UL1 + c] = R->f[F_U + c];
                R->f[F_U + c] = un;
                void* bs = R->f[F_BNL2 + c];
                R->f[F_BNL2 + c] = R->f[F_BNL1 + c];
                R->f[F_BNL1 + c] = R->f[F_BN + c];
                R->f[F_BN + c] = bs;
            }
            I[I_STEP] += 1;
            S[S_TIME] += S[S_DT];
        }
        break;
    }
    case FIN_POLL: {
        if (t == 0) {
            int v = 0;
            for (int c = 0; c < (a.ncomp > 1 ? a.ncomp : 1); ++c) v |= I[a.gate + c];
            a.host_flags[ri] = v;
        }
        break;
    }
    case FIN_SUM_RAW: {
        double s = slot_sum(R, a.f0, red);
        if (t == 0) S[S_RED + a.gate] = s;
        break;
    }
    case FIN_VOL: {
        double s = slot_sum(R, R_X3, red);
        if (t == 0) S[S_VOL] = s;
        break;
    }
    case FIN_STATS: {
        if (t == 0) {
            double* o = a.host_stats + (long long)ri * SEM_NSTAT;  // pinned host memory
            o[0] = S[S_TIME]; o[1] = S[S_KE]; o[2] = S[S_ENST]; o[3] = S[S_MAXDIV];
            for (int c = 0; c < 3; ++c) { o[4 + c] = I[I_VIT + c]; o[7 + c] = S[S_RN + c]; }
            o[10] = I[I_GIT]; o[11] = S[S_GBETA]; o[12] = I[I_NAN]; o[13] = I[I_STEP];
            o[14] = I[I_VREF] > I[I_VREF + 1] ? I[I_VREF] : I[I_VREF + 1];
            if (I[I_VREF + 2] > o[14]) o[14] = I[I_VREF + 2];
            o[15] = I[I_ORDER];
            o[16] = S[S_DT]; o[17] = S[S_CFL];
            o[18] = I[I_COMMIT];
        }
        break;
    }
    default: break;
    }
}


}  // namespace semk
