// One-dimensional contractions of lines held in registers (one line per
// thread) with a matrix that every thread of a wave reads alike: its rows come
// through scalar registers, RB rows a batch.  Scalar loads return in any order,
// so a wave waits for a whole batch; the address passes through asm so that a
// batch is loaded where it is asked for (hoisted ones spill).  A line costs its
// own LDS accesses only, instead of two LDS reads per multiply-add, and all
// sums ascend from zero, one fused multiply-add each.
#pragma once
#include "k_common.h"

namespace semk {

template <typename C> __device__ __forceinline__ void keep(C& v) { asm volatile("" : "+v"(v)); }

// row-major matrix of NC columns in device memory
template <int NC, typename C, int NB = 72 / (NC * (int)sizeof(C) / 4)> struct Rows {   // a batch: up to 72 scalar registers
    static constexpr int RB = NB;
    unsigned lo, hi;
    __device__ __forceinline__ void set(const void* p)
    {
        lo = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)p);
        hi = __builtin_amdgcn_readfirstlane((unsigned)((uintptr_t)p >> 32));
    }
    // rows r0 .. r0 + RB - 1 (zero from row n on)
    __device__ __forceinline__ void load(int r0, int n, C (&c)[RB][NC])
    {
        lo = __builtin_amdgcn_readfirstlane(lo);
        hi = __builtin_amdgcn_readfirstlane(hi);
        asm volatile("" : "+s"(lo), "+s"(hi)::"memory");
        typedef const __attribute__((address_space(4))) C* CP;
        const CP q = (CP)((uintptr_t)lo | ((uintptr_t)hi << 32)) + r0 * NC;
#pragma unroll
        for (int k = 0; k < RB; ++k)
#pragma unroll
            for (int a = 0; a < NC; ++a) c[k][a] = r0 + k < n ? q[k * NC + a] : (C)0;
    }
};

// out(o, sum_a mat[o][a] x[a]), o = 0 .. NR - 1
template <int NR, int NC, typename C, int RB, typename F>
__device__ __forceinline__ void rows_up(Rows<NC, C, RB> mat, const C (&x)[NC], F out)
{
#pragma unroll
    for (int o = 0; o < NR; o += RB) {
        C c[RB][NC], s[RB];
        mat.load(o, NR, c);
#pragma unroll
        for (int k = 0; k < RB; ++k) s[k] = 0;
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int k = 0; k < RB; ++k) s[k] = fma(c[k][a], x[a], s[k]);
#pragma unroll
        for (int k = 0; k < RB; ++k) keep(s[k]);
#pragma unroll
        for (int k = 0; k < RB; ++k)
            if (o + k < NR) out(o + k, s[k]);
    }
}
// y[a] = sum_o mat[o][a] in(o)
template <int NR, int NC, typename C, int RB, typename F>
__device__ __forceinline__ void rows_down(Rows<NC, C, RB> mat, F in, C (&y)[NC])
{
#pragma unroll
    for (int a = 0; a < NC; ++a) y[a] = 0;
#pragma unroll
    for (int o = 0; o < NR; o += RB) {
        C c[RB][NC];
        mat.load(o, NR, c);
#pragma unroll
        for (int k = 0; k < RB; ++k) {
            if (o + k >= NR) continue;
            const C v = in(o + k);
#pragma unroll
            for (int a = 0; a < NC; ++a) y[a] = fma(c[k][a], v, y[a]);
        }
#pragma unroll
        for (int a = 0; a < NC; ++a) keep(y[a]);
    }
}

}  // namespace semk
