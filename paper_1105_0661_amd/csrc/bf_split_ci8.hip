// bf_split_ci8.hip -- FP32 contraction of complex int8 samples on FP16 MFMAs.
#include "bf_split_worker.h"

namespace lbf {

hipError_t launch_split_ci8(const BlockDesc& d, hipStream_t st) { return launch_split_xt<XT_CI8>(d, st); }

}  // namespace lbf
