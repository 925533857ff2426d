// bf_fast_f32.hip -- fast contraction kernels with FP32 operands: the split
// worker (FP16 matrix instructions, FP32 results) for integer samples, FP32
// matrix instructions for complex float ones.
#include "bf_fast_impl.h"
#include "bf_split_worker.h"

namespace lbf {
hipError_t launch_fast_f32(const BlockDesc& d, hipStream_t st) {
    if (d.xtype == XT_CI8) return launch_split_ci8(d, st);
    if (d.xtype == XT_CI16) return launch_split_ci16(d, st);
    ItemGrid grid;
    const int n = block_items_fast_f32(d, &grid);
    return launch_f32(d, grid, n, st);
}
}  // namespace lbf
