#pragma once
// Helmholtz/Poisson operator on matrix cores for lx = 10..12 (N = 9..11):
//   w = h1 sum_ab D_a^T (G_ab o D_b u) + h2 B o u,  one wave per element.
//
// A wave holds its element's layers k as 16 x 16 tiles, rows j, columns i, in
// the accumulator layout of the 16x16x4 MFMA: lane (g = lane / 16, m = lane %
// 16) holds j = g + 4 r, i = m, r = 0..2.  Per layer:
//  - j-derivative  D U:    the tile as held is the B operand of step s (rows
//    j = 4 s + g), D the A operand, in registers for the whole kernel;
//  - i-derivative  U D^T:  U is the A operand, read transposed from the wave's
//    LDS;
//  - k-derivative: every lane holds whole columns, so it is a sum over the
//    layers in registers with uniform coefficients D[k][l];
//  - the six G_ab multiply point by point, and the transposed contractions
//    over i and j go through LDS into one chain of MFMA steps.
// MFMA adds its four products in ascending order, each with one rounding, so a
// chain of steps is the chain of fused multiply-adds of the column kernel
// (k_ax.hip).  The transposed contractions alternate i- and j-terms per index
// there; here the four products of a step are (l, i), (l, j), (l+1, i), (l+1,
// j).  Every result has the bits of the column kernel, which walked k with one
// thread per column and read 4 lx LDS values per point: LDS held it to 2.0 TB/s
// (three fp64 components, 16^3 elements, lx = 12: 363 us) and 1.5 TB/s in fp32.
// Here a tile of lx * lx points takes 18 LDS accesses of a wave.
//
// For fp32 the accumulator rows are 4 g + r; the rows of the A operand are
// permuted (row m holds j = m / 4 + 4 (m % 4)) so that the layout is the same.
#include "k_common.h"

#include <type_traits>

namespace semk {

template <typename C> struct WMma;
template <> struct WMma<double> {
    typedef double V4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V4 mma(double a, double b, V4 c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int arow(int m) { return m; }
};
template <> struct WMma<float> {
    typedef float V4 __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V4 mma(float a, float b, V4 c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int arow(int m) { return (m >> 2) + 4 * (m & 3); }
};

template <typename TG> struct AxwGeo {
    static constexpr int g = F_G16, b = F_B16;
};
template <> struct AxwGeo<double> {
    static constexpr int g = F_G64, b = F_B64;
};
template <> struct AxwGeo<float> {
    static constexpr int g = F_G32, b = F_B32;
};

// a value rounded to the 16-bit format H16 names (1 fp16, 2 bf16) and back
template <int H16, typename C> __device__ __forceinline__ C axw_r16(C x)
{
    if constexpr (H16 == 1) return (C)(float)(_Float16)(float)x;
    else if constexpr (H16 == 2) return (C)(float)(__bf16)(float)x;
    else return x;
}

// element c + off of a uniform array: a scalar base and a 32-bit lane offset, so
// that the many layers of a wave share their address registers
template <typename T> __device__ __forceinline__ const SEM_GLOBAL T* at(const SEM_GLOBAL T* base, int c, unsigned off)
{
    return (const SEM_GLOBAL T*)((const SEM_GLOBAL char*)(base + c) + (unsigned)(off * sizeof(T)));
}
template <typename T> __device__ __forceinline__ SEM_GLOBAL T* at(SEM_GLOBAL T* base, int c, unsigned off)
{
    return (SEM_GLOBAL T*)((SEM_GLOBAL char*)(base + c) + (unsigned)(off * sizeof(T)));
}

// Template parameters as ax_kernel (k_ax.hip): storage types of vectors TU and
// geometry TG, arithmetic C, PC Jacobi scaling of the input (1 fp64, 2 fp32
// diagonal), TW output, SUB residual form, H16 16-bit arithmetic, SHG geometry
// shared by the components through L2.
// Layers of G in flight (nb) and waves per SIMD that the registers must leave
// room for (mw).  fp64 holds 246 VGPRs with one layer; a second layer would
// cost the second wave (16^3, lx = 12: 209 us against 89).  fp32 at lx = 12:
// two layers at two waves 43 us, one layer at three waves 46; at lx = 10, with
// fewer points to a lane's registers, one layer at four waves 55 us against 57
// with two at two (20^3).  16-bit arithmetic keeps more operands: lx = 10 68 us
// at three waves, 80 at two; lx = 12 51 us at two, 54 at three.
template <int LX, typename C, int H16> struct AxwDepth {
    static constexpr int nb = sizeof(C) == 4 && !H16 && LX > 10 ? 2 : 1;
    static constexpr int mw = sizeof(C) == 8 || LX > 10 ? 2 : H16 ? 3 : 4;
};
template <int LX, int WPB, typename TU, typename TG, typename C, int PC, typename TW, int SUB = 0, int H16 = 0, int SHG = 0>
__global__ void __launch_bounds__(64 * WPB, (AxwDepth<LX, C, H16>::mw)) axw_kernel(Batch bt, AxLaunch a)
{
    using M = WMma<C>;
    typedef typename M::V4 V4;
    constexpr int EPB = WPB, L2 = LX * LX, L3 = L2 * LX;
    constexpr int NR = 3, KS = 3, KB = (LX + 1) / 2;
    constexpr int NCOL = (L2 * EPB + 63) / 64 * 64;  // columns of the block, as the partial sums group them
    constexpr int TS = 16 * LX + 16;                 // one tile in LDS, with room for the reads of unused lanes
    constexpr int SCR = 3 * TS, WS = SCR + 64;       // a wave's LDS: u, w_r, w_s, a slot per lane for unused stores
    static_assert(LX > 9 && LX <= 12, "three accumulator rows per lane");
    __shared__ __align__(16) C lds[EPB * WS];
    __shared__ C sD[H16 ? L2 : 1];
    __shared__ double red[NCOL / 64];
    static_assert(sizeof(double) * NCOL <= sizeof(C) * EPB * WS, "column dots reuse the tiles");

    // components of an element block on one XCD back to back, as ax_kernel
    const int bx = blockIdx.x;
    const int comp = (bx / 8) % a.ncomp;
    const int gb = (bx / (8 * a.ncomp)) * 8 + (bx & 7);
    const int* const pre = WPB == 1 ? bt.el : bt.eb;
    if (gb >= pre[bt.n]) return;
    const int ri = find_req(pre, bt.n, gb);
    const ReqDesc* R = bt.r[ri];
    const int blk = gb - pre[ri];
    if (!gate_ok(R, a.gate < 0 ? -1 : a.gate + comp)) return;

    const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63, g = lane >> 4, m = lane & 15;
    const int e = blk * EPB + w;
    const bool live = e < R->E;
    const int ee = live ? e : 0;  // a wave without an element works on element 0 and stores nothing
    if constexpr (H16 != 0) {
        for (int q = t; q < L2; q += 64 * EPB) sD[q] = axw_r16<H16>(gp(R->D32)[q]);
        block_sync_lds();
    }

    const SEM_GLOBAL TU* u = a.src_vj ? gfield<TU>(R, F_V) + (long long)gp(R->I)[I_GJ] * R->np
                                      : a.src >= 0 ? gfield<TU>(R, a.src + comp) : gp((const TU*)a.u_raw);
    SEM_GLOBAL TW* wo = a.dst >= 0 ? gfieldw<TW>(R, a.dst + comp) : gp((TW*)a.w_raw);
    using TPC = typename std::conditional<PC == 2, float, double>::type;
    C h1, h2;
    if (a.hsel >= 0) { h1 = (C)gp(R->S)[a.hsel]; h2 = (C)gp(R->S)[a.hsel + 1]; }
    else { h1 = (C)a.h1; h2 = (C)a.h2; }
    if (a.src_vj) h1 *= (C)gp(R->S)[S_GVS + gp(R->I)[I_GJ]];
    C gsc = (C)1, bsc = (C)1;
    const bool helm = h2 != (C)0;
    if constexpr (sizeof(TG) == 2) {
        const SEM_GLOBAL float* sc = gfield<float>(R, F_GSC);
        gsc = (C)sc[ee];
        bsc = (C)sc[R->E + ee];
    }
    const C gmul = H16 ? (C)1 : gsc;

    // the lane's three points of a layer: offsets in the element (unused lanes
    // and rows read an existing point of it) and in the LDS tile
    bool ok[NR];
    unsigned off[NR];
    int tix[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int j = g + 4 * r;
        ok[r] = m < LX && j < LX;
        off[r] = (j < LX ? j : LX - 1) * LX + (m < LX ? m : LX - 1);
        tix[r] = ok[r] ? j * LX + m : SCR + lane;
    }
    const SEM_GLOBAL TU* ue = u + (long long)ee * L3;
    const SEM_GLOBAL TG* Ge = gfield<TG>(R, AxwGeo<TG>::g) + (long long)ee * 6 * L3;
    const SEM_GLOBAL TG* Be = gfield<TG>(R, AxwGeo<TG>::b) + (long long)ee * L3;

    // all columns of u (and of the diagonal) and the first layer of G
    TU uraw[LX][NR];
    TPC praw[PC ? LX : 1][NR];
    constexpr int NB = AxwDepth<LX, C, H16>::nb;
    TG graw[NB][6][NR];
#pragma unroll
    for (int k = 0; k < LX; ++k)
#pragma unroll
        for (int r = 0; r < NR; ++r) uraw[k][r] = ldg(at(ue, k * L2, off[r]));
    const SEM_GLOBAL TPC* pe = PC ? gfield<TPC>(R, a.precond) + (long long)ee * L3 : nullptr;
    if constexpr (PC != 0) {
#pragma unroll
        for (int k = 0; k < LX; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r) praw[k][r] = ldg(at(pe, k * L2, off[r]));
    }
    auto gload = [&](int k) {
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                const SEM_GLOBAL TG* p = at(Ge, q * L3 + k * L2, off[r]);
                if constexpr (SHG != 0) graw[k % NB][q][r] = ldg(p);
                else graw[k % NB][q][r] = ldg_stream(p);
            }
    };
#pragma unroll
    for (int k = 0; k < NB; ++k) gload(k);

    // 1D matrices: cJ, cI (forward, rows j and columns i), cB (transposed: the
    // lane's index l of step s is 2 s + g / 2, even g an i-term, odd g a j-term)
    auto dmat = [&](int row, int col) -> C {
        if (row >= LX || col >= LX) return (C)0;
        if constexpr (sizeof(C) == 8) return (C)gp(R->D64)[row * LX + col];
        else return axw_r16<H16>((C)gp(R->D32)[row * LX + col]);
    };
    const int mj = M::arow(m);
    C cJ[KS], cI[KS], cB[KB];
#pragma unroll
    for (int s = 0; s < KS; ++s) { cJ[s] = dmat(mj, 4 * s + g); cI[s] = dmat(m, 4 * s + g); }
    const bool jterm = (g & 1) != 0;
#pragma unroll
    for (int s = 0; s < KB; ++s) cB[s] = dmat(2 * s + (g >> 1), jterm ? mj : m);
    C* const st = lds + w * WS;
    const int ubase = mj * LX + g;
    const int bbase = jterm ? 2 * TS + (g >> 1) * LX + m : TS + mj * LX + (g >> 1);
    const int bstep = jterm ? 2 * LX : 2;

    C ureg[LX][NR], wacc[LX][NR];
#pragma unroll
    for (int k = 0; k < LX; ++k)
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            C v = to<C>(uraw[k][r]);
            if constexpr (PC != 0) v *= (C)praw[k][r];
            if (LX % 4 != 0 && r == NR - 1) v = g + 4 * r < LX ? v : (C)0;  // rows past the element add nothing
            ureg[k][r] = v;
            wacc[k][r] = (C)0;
        }
    C hscale = (C)1;
    if constexpr (H16 != 0) {
        float mx = 0.0f;
#pragma unroll
        for (int k = 0; k < LX; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r) mx = fmaxf(mx, ok[r] ? fabsf((float)ureg[k][r]) : 0.0f);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        float sc = 1.0f;
        if (mx > 0.0f && mx < INFINITY) {
            int ex;
            (void)frexpf(mx, &ex);
            sc = ldexpf(1.0f, -ex);
        }
        hscale = (C)(1.0f / sc);
#pragma unroll
        for (int k = 0; k < LX; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r) ureg[k][r] = axw_r16<H16>(ureg[k][r] * sc);
    }

    // uniform coefficients D[k][.]: scalar loads (the table does not change)
    typedef const __attribute__((address_space(4))) C* CP;
    const uintptr_t dp = sizeof(C) == 8 ? (uintptr_t)R->D64 : (uintptr_t)R->D32;
    unsigned dlo = __builtin_amdgcn_readfirstlane((unsigned)dp), dhi = __builtin_amdgcn_readfirstlane((unsigned)(dp >> 32));

#pragma unroll
    for (int k = 0; k < LX; ++k) {
#pragma unroll
        for (int r = 0; r < NR; ++r) st[tix[r]] = ureg[k][r];
        // (keeps each layer's coefficients from being loaded ahead of it)
        asm volatile("" : "+s"(dlo), "+s"(dhi));
        const CP Dt = (CP)((uintptr_t)dlo | ((uintptr_t)dhi << 32));
        C dk[LX];
#pragma unroll
        for (int l = 0; l < LX; ++l) dk[l] = H16 ? sD[H16 ? k * LX + l : 0] : Dt[k * LX + l];
        lds_handoff<true>();
        C ut_[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            ut_[s] = st[ubase + 4 * s];
            if (LX % 4 != 0 && s == KS - 1) ut_[s] = 4 * s + g < LX ? ut_[s] : (C)0;
        }
        V4 ur = {0, 0, 0, 0}, us = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            us = M::mma(cJ[s], ureg[k][s], us);
            ur = M::mma(ut_[s], cI[s], ur);
        }
        C wt[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            C ut = 0;
#pragma unroll
            for (int l = 0; l < LX; ++l) ut += dk[l] * ureg[l][r];
            C g6[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) g6[q] = to<C>(graw[k % NB][q][r]) * gmul;
            const C wr = axw_r16<H16>(g6[0] * ur[r] + g6[1] * us[r] + g6[2] * ut);
            const C ws = axw_r16<H16>(g6[1] * ur[r] + g6[3] * us[r] + g6[4] * ut);
            wt[r] = axw_r16<H16>(g6[2] * ur[r] + g6[4] * us[r] + g6[5] * ut);
            st[TS + tix[r] - (ok[r] ? 0 : TS)] = wr;
            st[2 * TS + tix[r] - (ok[r] ? 0 : 2 * TS)] = ws;
        }
        if (k + NB < LX) gload(k + NB);
#pragma unroll
        for (int l = 0; l < LX; ++l)
#pragma unroll
            for (int r = 0; r < NR; ++r) wacc[l][r] += dk[l] * wt[r];
        lds_handoff<true>();
        V4 acc = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KB; ++s) {
            C v = st[bbase + s * bstep];
            if (LX % 2 != 0 && s == KB - 1) v = 2 * s + (g >> 1) < LX ? v : (C)0;
            acc = M::mma(jterm ? cB[s] : v, jterm ? v : cB[s], acc);
        }
#pragma unroll
        for (int r = 0; r < NR; ++r) wacc[k][r] += acc[r];
        // the layer's sums are formed here, not kept as operands for later,
        // and the lane offsets stay 32-bit operands of scalar-base loads
#pragma unroll
        for (int l = 0; l < LX; ++l)
#pragma unroll
            for (int r = 0; r < NR; ++r) asm volatile("" : "+v"(wacc[l][r]));
#pragma unroll
        for (int r = 0; r < NR; ++r) asm volatile("" : "+v"(off[r]));
    }

    double dot[NR] = {0.0, 0.0, 0.0};
    const C hs = H16 ? h1 * (gsc * hscale) : h1;
    const SEM_GLOBAL TW* rl = SUB ? gfield<TW>(R, a.sub + comp) + (long long)ee * L3 : nullptr;
    SEM_GLOBAL TW* we = wo + (long long)ee * L3;
    // the mass term and the local rhs are loaded only now, half the layers at a
    // time: through the k-walk their registers would cost the second wave
    constexpr int HB = (LX + 1) / 2;
#pragma unroll
    for (int k0 = 0; k0 < LX; k0 += HB) {
        TG braw[HB][NR];
        TW rraw[SUB ? HB : 1][NR];
        // 16-bit arithmetic: the input as stored again (the registers hold its
        // scaled rounding)
        TU urd[H16 ? HB : 1][NR];
        TPC prd[H16 && PC ? HB : 1][NR];
        if constexpr (H16 != 0) {
#pragma unroll
            for (int k = 0; k < HB; ++k)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (k0 + k < LX) {
                        urd[k][r] = ldg(at(ue, (k0 + k) * L2, off[r]));
                        if constexpr (PC != 0) prd[k][r] = ldg(at(pe, (k0 + k) * L2, off[r]));
                    }
        }
        if (helm) {
#pragma unroll
            for (int k = 0; k < HB; ++k)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (k0 + k < LX) braw[k][r] = ldg(at(Be, (k0 + k) * L2, off[r]));
        }
        if constexpr (SUB != 0) {
#pragma unroll
            for (int k = 0; k < HB; ++k)
#pragma unroll
                for (int r = 0; r < NR; ++r)
                    if (k0 + k < LX) rraw[k][r] = ldg(at(rl, (k0 + k) * L2, off[r]));
        }
#pragma unroll
        for (int k = 0; k < HB; ++k)
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                if (k0 + k >= LX) continue;
                const int kk = k0 + k;
                C uk = ureg[kk][r];
                if constexpr (H16 != 0) {
                    uk = to<C>(urd[k][r]);
                    if constexpr (PC != 0) uk *= (C)prd[k][r];
                }
                const C bk = helm ? to<C>(braw[k][r]) * bsc : (C)0;
                const C wv = hs * wacc[kk][r] + h2 * bk * uk;
                const TW ws = SUB ? (TW)(rraw[SUB ? k : 0][r] - to<TW>(wv)) : to<TW>(wv);
                if (live && ok[r]) stg(at(we, kk * L2, off[r]), ws);
                if (a.pdot >= 0) dot[r] += (double)uk * (double)to<C>(ws);
            }
    }
    if (a.pdot >= 0 && a.dots >= 0) {
        // the columns' dots, for axw_dots_kernel
        SEM_GLOBAL double* cd = gfieldw<double>(R, a.dots + comp) + (long long)ee * L2;
#pragma unroll
        for (int r = 0; r < NR; ++r)
            if (live && ok[r]) cd[off[r]] = dot[r];
    } else if (a.pdot >= 0) {
        // the columns' dots, summed in the order of the column kernel's threads
        double* cd = (double*)lds;
        block_sync_lds();
        for (int q = EPB * L2 + t; q < NCOL; q += 64 * EPB) cd[q] = 0.0;
#pragma unroll
        for (int r = 0; r < NR; ++r)
            if (ok[r]) cd[w * L2 + off[r]] = live ? dot[r] : 0.0;
        block_sync_lds();
        for (int q = w; q < NCOL / 64; q += EPB) {
            const double s = wave_sum(cd[64 * q + lane]);
            if (lane == 0) red[q] = s;
        }
        block_sync_lds();
        if (t == 0) {
            double s = 0.0;
            for (int q = 0; q < NCOL / 64; ++q) s += red[q];
            gp(R->part)[(long long)(a.pdot + comp) * R->pstride + blk] = s;
            if (blk == 0) gp(R->I)[I_PCNT + a.pdot + comp] = R->nb;
        }
    }
}

// the partial sums of the column dots of an element block, in the order in
// which axw_kernel adds them itself
template <int LX>
__global__ void __launch_bounds__((epb_of(LX) * LX * LX + 63) / 64 * 64) axw_dots_kernel(Batch bt, AxLaunch a)
{
    constexpr int EPB = epb_of(LX), L2 = LX * LX, NW = (EPB * L2 + 63) / 64;
    __shared__ double red[NW];
    const int comp = blockIdx.y, g = blockIdx.x;
    const int ri = find_req(bt.eb, bt.n, g);
    const ReqDesc* R = bt.r[ri];
    if (!gate_ok(R, a.gate < 0 ? -1 : a.gate + comp)) return;
    const int blk = g - bt.eb[ri], t = threadIdx.x;
    const long long q = (long long)blk * EPB * L2 + t;
    const SEM_GLOBAL double* cd = gfield<double>(R, a.dots + comp);
    const double s = wave_sum(t < EPB * L2 && q < (long long)R->E * L2 ? cd[q] : 0.0);
    if ((t & 63) == 0) red[t >> 6] = s;
    block_sync_lds();
    if (t == 0) {
        double v = 0.0;
        for (int w = 0; w < NW; ++w) v += red[w];
        gp(R->part)[(long long)(a.pdot + comp) * R->pstride + blk] = v;
        if (blk == 0) gp(R->I)[I_PCNT + a.pdot + comp] = R->nb;
    }
}

// Without the fused dot a wave is a workgroup of its own.  With it the
// workgroups are the element blocks its partial sums are defined on, except
// where these hold more than two waves and do not run in one round: then the
// waves still run alone and leave their column dots in the scratch field a.dots.
// At lx = 10 a CU holds three blocks of five fp32 waves or one of fp64, where 16
// and eight waves fit.  Three components and their dots, us, blocks against single
// waves: 1440 elements (864 blocks) fp32 49.5 / 38.0, fp64 84.7 / 67.9 (column
// kernel 46.4, 96.5).  Up to 768 blocks the three of a CU run in one round (1280
// elements, fp32: blocks 35.5, column kernel 37.2).
template <int LX, typename TU, typename TG, typename C, int H16 = 0>
static void axw_go(const Batch& b, const AxLaunch& a0, hipStream_t s)
{
    constexpr int EPB = epb_of(LX);
    // 16-bit arithmetic at lx = 10 comes here neither scaled nor with the dot (ax_wide)
    constexpr bool ALONE = LX == 10 && H16 != 0;
    AxLaunch a = a0;
    if (a.pdot >= 0 && (EPB <= 2 || b.eb[b.n] * a.ncomp <= 768)) a.dots = -1;
    const bool blocks = a.pdot >= 0 && a.dots < 0;
    const int n = blocks ? b.eb[b.n] : b.el[b.n];
    const dim3 grid(((n + 7) / 8) * 8 * a.ncomp);
#define AXW_GO(W, ...) hipLaunchKernelGGL((axw_kernel<LX, W, TU, TG, C, __VA_ARGS__>), grid, dim3(64 * W), 0, s, b, a)
    if constexpr (sizeof(TU) == 4) {
        // the Arnoldi operator of an fp32 GMRES basis
        if (a.out64) {
            if constexpr (!ALONE) {
                if (a.precond >= 0 && a.tpc == P64) { AXW_GO(1, 1, double, 0, H16); return; }
                if (a.precond >= 0) { AXW_GO(1, 2, double, 0, H16); return; }
            }
            AXW_GO(1, 0, double, 0, H16);
            return;
        }
    }
    if constexpr (sizeof(TU) == 8) {
        // the Arnoldi operator of an fp64 GMRES basis
        if (a.precond >= 0 && a.tpc == P64) { AXW_GO(1, 1, TU, 0, H16); return; }
        if (a.precond >= 0) { AXW_GO(1, 2, TU, 0, H16); return; }
    }
    if constexpr (sizeof(TU) == 8 && sizeof(TG) == 8 && sizeof(C) == 8 && H16 == 0) {
        if (a.sub >= 0) {
            if (a.ncomp > 1) AXW_GO(1, 0, TU, 1, 0, 1);
            else AXW_GO(1, 0, TU, 1);
            return;
        }
    }
    if constexpr (!ALONE) {
        if (blocks) {
            if (a.ncomp > 1) AXW_GO(EPB, 0, TU, 0, H16, 1);
            else AXW_GO(EPB, 0, TU, 0, H16);
            return;
        }
    }
    if (a.ncomp > 1) AXW_GO(1, 0, TU, 0, H16, 1);
    else AXW_GO(1, 0, TU, 0, H16);
    if (a.pdot >= 0)
        hipLaunchKernelGGL(axw_dots_kernel<LX>, dim3(b.eb[b.n], a.ncomp), dim3((EPB * LX * LX + 63) / 64 * 64), 0, s, b, a);
#undef AXW_GO
}

// the (vector, geometry, arithmetic) combinations of ax_lx (k_ax.hip)
template <int LX> static void axw_lx(const Batch& b, const AxLaunch& a, hipStream_t s)
{
    const int u = a.tu, g = a.tg, c = a.tc;
    if (u == P64 && g == P64 && c == P64) axw_go<LX, double, double, double>(b, a, s);
    else if (u == P64 && g == P32 && c == P64) axw_go<LX, double, float, double>(b, a, s);
    else if (u == P64 && g == P16 && c == P64) axw_go<LX, double, __half, double>(b, a, s);
    else if (u == P64 && g == PBF && c == P64) axw_go<LX, double, __hip_bfloat16, double>(b, a, s);
    else if (u == P64 && g == P32 && c == P32) axw_go<LX, double, float, float>(b, a, s);
    else if (u == P64 && g == P16 && c == P32) axw_go<LX, double, __half, float>(b, a, s);
    else if (u == P64 && g == PBF && c == P32) axw_go<LX, double, __hip_bfloat16, float>(b, a, s);
    else if (u == P32 && g == P32 && c == P64) axw_go<LX, float, float, double>(b, a, s);
    else if (u == P32 && g == P16 && c == P64) axw_go<LX, float, __half, double>(b, a, s);
    else if (u == P32 && g == PBF && c == P64) axw_go<LX, float, __hip_bfloat16, double>(b, a, s);
    else if (u == P32 && g == P32 && c == P32) axw_go<LX, float, float, float>(b, a, s);
    else if (u == P32 && g == P16 && c == P32) axw_go<LX, float, __half, float>(b, a, s);
    else if (u == P32 && g == PBF && c == P32) axw_go<LX, float, __hip_bfloat16, float>(b, a, s);
    else if (u == P16 && g == P16 && c == P32) axw_go<LX, __half, __half, float>(b, a, s);
    else if (u == PBF && g == PBF && c == P32) axw_go<LX, __hip_bfloat16, __hip_bfloat16, float>(b, a, s);
    // 16-bit arithmetic: at lx = 11 the column kernel's LDS reads fall in
    // different banks and it is faster (18^3: 57 us against 67)
    if constexpr (LX != 11) {
        if (u == P32 && g == P16 && c == P16) axw_go<LX, float, __half, float, 1>(b, a, s);
        else if (u == P16 && g == P16 && c == P16) axw_go<LX, __half, __half, float, 1>(b, a, s);
        else if (u == P32 && g == PBF && c == PBF) axw_go<LX, float, __hip_bfloat16, float, 2>(b, a, s);
        else if (u == PBF && g == PBF && c == PBF) axw_go<LX, __hip_bfloat16, __hip_bfloat16, float, 2>(b, a, s);
    }
}

}  // namespace semk
