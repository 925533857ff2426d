// bf_split_ci16.hip -- FP32 contraction of complex int16 samples on FP16 MFMAs.
#include "bf_split_worker.h"

namespace lbf {

hipError_t launch_split_ci16(const BlockDesc& d, hipStream_t st) { return launch_split_xt<XT_CI16>(d, st); }

}  // namespace lbf
