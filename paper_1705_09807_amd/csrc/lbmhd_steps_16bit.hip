// Multi-step sweeps (lbmhd_steps.h) for FP16 and BF16 storage, and the dispatch on the
// storage type.
#include "lbmhd_steps.h"

namespace lbm {

hipError_t launch_steps_fp64(const Launch& L, int k);
hipError_t launch_steps_fp32(const Launch& L, int k);

hipError_t launch_steps(const Launch& L, int k) {
  switch (L.dtype) {
    case LBM_FP64: return launch_steps_fp64(L, k);
    case LBM_FP32: return launch_steps_fp32(L, k);
    case LBM_FP16: return launch_steps_typed<_Float16>(L, k);
    default: return launch_steps_typed<__bf16>(L, k);
  }
}

}  // namespace lbm
