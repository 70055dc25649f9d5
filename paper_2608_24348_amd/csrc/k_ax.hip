// The Helmholtz operator: choice of the kernel, and the column kernel at
// lx = 3..7 (the other orders have sources of their own: the forms of one order
// take about a minute to compile).
#include "k_ax.h"

namespace semk {

// The matrix-core operator of lx = 10..12 (k_axw.h) gives a wave an element,
// the column kernel an element to two or three waves.  Each runs in rounds, so
// the rule counts workgroups a CU of the column kernel (wg: it holds one at a
// time at lx = 10 and 12, two at lx = 11) and waves a SIMD of the matrix-core
// kernel (waves).  us, column kernel / matrix cores:
//   lx = 12: past the first round.  512 elements (wg 1) fp64 16.0 / 17.4, fp32
//     10.9 / 12.5; 640 (wg 2) 29.0 / 18.9; 16^3 127 / 94, fp32 77 / 43
//   lx = 11, fp64 arithmetic: past two (1280 elements, wg 3, 31.0 / 25.9).  With
//     the Jacobi scaling and fp64 geometry the extra registers leave a launch of
//     many waves at par, and behind where the column kernel's last round is full:
//     2560 elements (wg 5, waves 3) 54.4 / 57.1, 3584 (wg 7, waves 4) 4% slower
//   lx = 11, fp32 arithmetic: past three: a third workgroup alone on its CU is
//     soon done (1440 elements, wg 3, 16.0 / 17.4; fp16 geometry 15.6 / 18.2),
//     a fourth is not (1728 22.7 / 18.3).  fp16 vectors, whose conversions weigh
//     more: only while two waves a SIMD hold the launch (1728 elements 0.87 of
//     the column kernel's time, 2560 1.16, 3584 1.07, 5832 1.02)
//   lx = 10: past the first round (1728 elements fp32 19.7 / 15.7, 20^3 69 / 57),
//     but with 16-bit geometry not at two full rounds against three waves (2560
//     elements, fp16 vectors 20.2 / 22.7, fp32 20.6 / 21.5).  fp64 arithmetic is on matrix
//     cores at every size (8 elements 18.4 / 12.2): rows of ten doubles fall in
//     the same LDS banks
//   16-bit arithmetic: lx = 11 stays with the column kernel (18^3: 57 / 67).  lx =
//     10: alone, while its waves do not outnumber the column kernel's rounds (1440
//     to 2048 elements 0.90 of its time, 3072 0.82; 2560 1.14, 3584 1.15); not
//     with the fused dot (three components, 512 to 1920 elements 1.26 to 1.39,
//     above 0.94 to 1.03) nor with the Jacobi scaling (0.91 to 1.14)
// lx = 9 has no bank conflicts and would leave two thirds of a 16 x 16 tile empty
// (22^3: fp64 138 / 145, fp32 66 / 71).  Both kernels give the same bits.
static bool ax_wide(const Batch& b, int lx, const AxLaunch& a)
{
    if (lx < 10 || lx > 12) return false;
    const bool half = a.tc == P16 || a.tc == PBF;
    if (lx == 10 && a.tc == P64) return true;
    if (lx == 11 && half) return false;
    const int wg = (b.eb[b.n] * a.ncomp + 255) / 256, waves = (b.el[b.n] * a.ncomp + 1023) / 1024;
    if (lx == 12) return wg > 1;
    if (lx == 11) {
        if (a.tc == P64) return wg > 2 && !(a.tg == P64 && a.precond >= 0 && waves > 2 && wg < 2 * waves);
        return wg > 3 && !(a.tu == P16 && waves > 2);
    }
    if (half) return wg > 1 && waves <= wg && a.precond < 0 && a.pdot < 0;
    return wg > 1 && !(wg == 2 && waves > 2 && a.tg != P32);
}

void launch_ax(const Batch& b, int lx, const AxLaunch& a0, hipStream_t s)
{
    AxLaunch a = a0;
    if (a.ncomp < 1) a.ncomp = 1;
    if (launch_ax_mfma(b, lx, a, s)) return;
    const bool wide = ax_wide(b, lx, a);
    switch (lx) {
    case 3: ax_lx<3>(b, a, s); break;
    case 4: ax_lx<4>(b, a, s); break;
    case 5: ax_lx<5>(b, a, s); break;
    case 6: ax_lx<6>(b, a, s); break;
    case 7: ax_lx<7>(b, a, s); break;
    case 8: launch_ax_col8(b, a, s); break;
    case 9: launch_ax_col9(b, a, s); break;
    case 10: wide ? launch_ax_wide10(b, a, s) : launch_ax_col10(b, a, s); break;
    case 11: wide ? launch_ax_wide11(b, a, s) : launch_ax_col11(b, a, s); break;
    case 12: wide ? launch_ax_wide12(b, a, s) : launch_ax_col12(b, a, s); break;
    default: break;
    }
}

}  // namespace semk
