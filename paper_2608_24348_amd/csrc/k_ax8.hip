// The column Helmholtz operator at lx = 8 and 9.
#include "k_ax.h"

namespace semk {

void launch_ax_col8(const Batch& b, const AxLaunch& a, hipStream_t s) { ax_lx<8>(b, a, s); }
void launch_ax_col9(const Batch& b, const AxLaunch& a, hipStream_t s) { ax_lx<9>(b, a, s); }

}  // namespace semk
