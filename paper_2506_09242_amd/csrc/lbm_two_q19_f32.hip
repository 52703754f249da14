// Two-step kernels, D3Q19, precision f32 (lbm_prec 1).
#include "lbm_two.h"

namespace lbmd {
template hipError_t launch_two_steps<19, 1>(const StepParams &, void *, const TwoTiles &, int, bool, int, hipStream_t);
}  // namespace lbmd
