// MFMA kernel instances: fp32 basis operands, with the workspace rows, one robot tile.
#include "sf_fast_kernel.h"

namespace sf {

hipError_t fast_single_p0_w1_r1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int W) {
  return fastk::launch_single_mp<0, 1, 1>(p, a, tab32, a16, W);
}

hipError_t fast_class_p0_w1_r1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int ci, int grid, int W) {
  return fastk::launch_batched_mp<0, 1, 1>(p, a, tab32, a16, ci, grid, W);
}

hipError_t fast_segments_p0_w1_r1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16) {
  return fastk::launch_segments_mp<0, 1, 1>(p, a, tab32, a16);
}

}  // namespace sf
