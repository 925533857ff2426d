// bf_split_cf32.hip -- FP32 contraction of complex float samples on FP16 MFMAs.
#include "bf_split_worker.h"

namespace lbf {

hipError_t launch_split_cf32(const BlockDesc& d, hipStream_t st) { return launch_split_xt<XT_CF32>(d, st); }

}  // namespace lbf
