// bf_fast_bf16_cf32.hip -- fast contraction kernels with BF16 operands, complex float samples.
#include "bf_fast_impl.h"

namespace lbf {
hipError_t launch_bf16_cf32(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    return launch_h_xt<XT_CF32, CT_BF16>(d, grid, n, st);
}
}  // namespace lbf
