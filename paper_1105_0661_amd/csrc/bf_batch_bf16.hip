// bf_batch_bf16.hip -- persistent batch kernels with BF16 operands.
#include "bf_batch_impl.h"

namespace lbf {
hipError_t launch_batch_bf16(int v, const BatchArgs& a, int* counter, hipStream_t st) {
    return launch_batch_variant<CT_BF16>(v, a, counter, st);
}
}  // namespace lbf
