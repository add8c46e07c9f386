// Evaluation kernel instantiations: 16 lanes per evaluation, 1 copy splitting the cuboids.
#include "mg_eval_lane.h"

namespace mg {
hipError_t launch_eval_l16h1(const EvalArgs& a, int grid_x, bool cand, bool grad, hipStream_t s) {
  return launch_eval_shape<16, 1>(a, grid_x, cand, grad, s);
}
}  // namespace mg
