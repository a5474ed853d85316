// Multi-step sweeps (lbmhd_steps.h) for FP64 storage.
#include "lbmhd_steps.h"

namespace lbm {

hipError_t launch_steps_fp64(const Launch& L, int k) { return launch_steps_typed<double>(L, k); }

}  // namespace lbm
