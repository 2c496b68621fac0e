// MFMA kernel instances: bf16 basis operands, with the workspace rows, one robot tile.
#include "sf_fast_kernel.h"

namespace sf {

hipError_t fast_single_p1_w1_r1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int W) {
  return fastk::launch_single_mp<1, 1, 1>(p, a, tab32, a16, W);
}

hipError_t fast_class_p1_w1_r1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int ci, int grid, int W) {
  return fastk::launch_batched_mp<1, 1, 1>(p, a, tab32, a16, ci, grid, W);
}

}  // namespace sf
