// bf_fast_f16_cf32.hip -- fast contraction kernels with F16 operands, complex float samples.
#include "bf_fast_impl.h"

namespace lbf {
hipError_t launch_f16_cf32(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    return launch_h_xt<XT_CF32, CT_F16>(d, grid, n, st);
}
}  // namespace lbf
