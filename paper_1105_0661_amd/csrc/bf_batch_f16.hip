// bf_batch_f16.hip -- persistent batch kernels with F16 operands.
#include "bf_batch_impl.h"

namespace lbf {
hipError_t launch_batch_f16(int v, const BatchArgs& a, int* counter, hipStream_t st) {
    return launch_batch_variant<CT_F16>(v, a, counter, st);
}
}  // namespace lbf
