// Two-step kernels, D3Q19, precision f64 (lbm_prec 0).
#include "lbm_two.h"

namespace lbmd {
template hipError_t launch_two_steps<19, 0>(const StepParams &, void *, const TwoTiles &, int, bool, int, hipStream_t);
}  // namespace lbmd
