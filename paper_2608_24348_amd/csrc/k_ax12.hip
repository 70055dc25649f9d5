// The column Helmholtz operator at lx = 12.
#include "k_ax.h"

namespace semk {

void launch_ax_col12(const Batch& b, const AxLaunch& a, hipStream_t s) { ax_lx<12>(b, a, s); }

}  // namespace semk
