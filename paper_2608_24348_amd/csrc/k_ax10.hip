// The column Helmholtz operator at lx = 10 and 11.
#include "k_ax.h"

namespace semk {

void launch_ax_col10(const Batch& b, const AxLaunch& a, hipStream_t s) { ax_lx<10>(b, a, s); }
void launch_ax_col11(const Batch& b, const AxLaunch& a, hipStream_t s) { ax_lx<11>(b, a, s); }

}  // namespace semk
