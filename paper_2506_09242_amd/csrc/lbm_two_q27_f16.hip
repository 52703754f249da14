// Two-step kernels, D3Q27, precision f16 (lbm_prec 2).
#include "lbm_two.h"

namespace lbmd {
template hipError_t launch_two_steps<27, 2>(const StepParams &, void *, const TwoTiles &, int, bool, int, hipStream_t);
}  // namespace lbmd
