// Multi-step sweeps (lbmhd_steps.h) for FP32 storage.
#include "lbmhd_steps.h"

namespace lbm {

hipError_t launch_steps_fp32(const Launch& L, int k) { return launch_steps_typed<float>(L, k); }

}  // namespace lbm
