// The matrix-core Helmholtz/Poisson operator at lx = 11 (a source of its own per
// order: the forms of one take minutes to compile).
#include "k_axw.h"

namespace semk {

void launch_ax_wide11(const Batch& b, const AxLaunch& a, hipStream_t s) { axw_lx<11>(b, a, s); }

}  // namespace semk
