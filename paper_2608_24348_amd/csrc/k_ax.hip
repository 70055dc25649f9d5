// The Helmholtz operator: choice of the kernel, and the column kernel at
// lx = 3..7 (the other orders have sources of their own: the forms of one order
// take about a minute to compile).
#include "k_ax.h"

namespace semk {

// The matrix-core operator of lx = 10..12 (k_axw.h) gives a wave an element,
// the column kernel an element to two or three waves, so a launch that the
// column kernel finishes in one round of the 256 CUs stays there (it holds one
// workgroup to a CU at lx = 10 and 12, two at lx = 11).  Beyond that round, in
// us, column kernel against matrix cores:
//   lx = 12, fp64  512 elements 16.0 / 17.4, 1000 30.9 / 21.8, 16^3 127 / 94
//            fp32  512 10.9 / 12.5, 1000 20.3 / 14.6, 16^3 77 / 43
//   lx = 11, fp64  1000 19.5 / 20.6, 1728 37.2 / 33.1; fp32 1728 22.7 / 18.3
//   lx = 10, fp32  1000 10.6 / 12.7, 1728 19.7 / 15.7, 20^3 69 / 57
// fp64 at lx = 10 is on matrix cores at every size (8 elements 18.4 / 12.2):
// rows of ten doubles fall in the same LDS banks.  16-bit arithmetic at lx = 11
// stays with the column kernel (18^3: 57 / 67).  lx = 9 has no such conflicts
// and would leave two thirds of a 16 x 16 tile empty (22^3: fp64 138 / 145,
// fp32 66 / 71).  Both kernels give the same bits.
static bool ax_wide(const Batch& b, int lx, const AxLaunch& a)
{
    if (lx < 10 || lx > 12) return false;
    const bool half = a.tc == P16 || a.tc == PBF;
    if (lx == 10 && a.tc == P64) return true;
    if (lx == 11 && half) return false;
    return b.eb[b.n] * a.ncomp > (lx == 11 ? 512 : 256);
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
