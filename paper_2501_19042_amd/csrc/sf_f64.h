// FP64 matrix-core path of the safety filter (2D and 3D swarms of up to 32 robots): launch interface.
#pragma once

#include "sf_internal.h"

namespace sf {

// Whether the FP64 matrix-core kernels cover a config: up to 32 robots, degree <= 15, horizon <= 256 and
// an LDS plan within 160 KB.
bool f64_cfg_covered(const DevCfg& c);
// Doubles of the basis-operand table of one config, and its contents: [tile][basis][S1 A operand, S4 B
// operand (x rho)][lane][4].
int64_t a64_entries(const DevCfg& c);
void a64_fill(const DevCfg& c, const double* P3, double* out);
// Waves per sample for a batch of these configs with R robot tiles of 16, and its LDS bytes; 0: it does
// not fit, or its units are out of the range of fp32 drift bounds.  The solve over the batch's work items;
// a.tab the FP64 factor table, D the configs' dimensions.
int f64_waves(const DevCfg* const* cfgs, int n_cfgs, int R, int64_t n_items, int ncu, size_t* lds);
hipError_t launch_f64_project(const LaunchArgs& a, const double* a64, int D, int R, int W);

// FP64 feasibility check of a batch of covered configs (violations as in launch_feasibility).
struct CheckArgs {
  const DevCfg* cfgs;
  const double* tab;
  const double* a64;
  const DevProblem* probs;
  const WorkItem* items;
  int32_t n_items;
  const void* xi;
  const void* bvals;
  double* viol;
  size_t lds_bytes;
  hipStream_t stream;
};
size_t f64_check_lds_bytes(const DevCfg& c, int R);
hipError_t launch_f64_check(const CheckArgs& a, bool dbl, int D, int R);

}  // namespace sf
