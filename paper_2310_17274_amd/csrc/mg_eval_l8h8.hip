// Evaluation kernel instantiations: 8 lanes per evaluation, 8 copies splitting the cuboids.
#include "mg_eval_lane.h"

namespace mg {
hipError_t launch_eval_l8h8(const EvalArgs& a, int grid_x, bool cand, bool grad, hipStream_t s) {
  return launch_eval_shape<8, 8>(a, grid_x, cand, grad, s);
}
}  // namespace mg
