// MFMA kernel instances: bf16 basis operands, with the workspace rows.
#include "sf_fast_kernel.h"

namespace sf {

hipError_t fast_launch_single_p1_w1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16,
                                     int W) {
  return fastk::launch_single_mp<1, 1>(p, a, tab32, a16, W);
}

hipError_t fast_launch_batched_p1_w1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16,
                                      const int* grid, const int* W, int cls_mask) {
  return fastk::launch_batched_mp<1, 1>(p, a, tab32, a16, grid, W, cls_mask);
}

hipError_t fast_launch_segments_p1_w1(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16) {
  return fastk::launch_segments_mp<1, 1>(p, a, tab32, a16);
}

}  // namespace sf
