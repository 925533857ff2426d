// bf_fast_bf16_ci16.hip -- fast contraction kernels with BF16 operands, complex int16 samples.
#include "bf_fast_impl.h"

namespace lbf {
hipError_t launch_bf16_ci16(const BlockDesc& d, const ItemGrid& grid, int n, hipStream_t st) {
    return launch_h_xt<XT_CI16, CT_BF16>(d, grid, n, st);
}
}  // namespace lbf
