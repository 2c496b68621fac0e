// Adjoint (reverse-mode) kernel of the unrolled safety-filter iterations.
#pragma once

#include "sf_internal.h"

namespace sf {

struct AdjointArgs {
  const DevCfg* cfgs;
  const void* tab;
  const DevProblem* probs;
  const WorkItem* items;
  int32_t n_items;
  const void* xi_bar;
  const void* bvals;
  int32_t iters;
  const void* ckpt;
  int32_t ckpt_every;
  int64_t ckpt_stride;
  const void* g_xi_out;
  const void* g_lam_out;
  const void* g_resid;
  const void* w_fpr;            // [S] cotangent of the fixed-point residual sum, or NULL
  void* g_xi0;
  void* g_lam0;
  void* g_xi_bar;
  void* states;                 // scratch: n_items * state_stride elements
  int64_t state_stride;         // 2 (ckpt_every + 1) * largest n * D * m of the batch (xi, then lambda)
  int32_t tile;
  size_t lds_bytes;
  hipStream_t stream;
};

template <typename T>
hipError_t launch_adjoint(const AdjointArgs& a);

size_t adjoint_lds_bytes(const DevCfg& c, int tile, size_t elem);

// MFMA adjoint path (fp32; 3D, up to 32 robots, degree <= 15, horizon <= 256).  The forward states of one or
// more checkpoint segments are recomputed by the forward MFMA kernel into `states` ([segment - seg0][every +
// 1][2][stride], stride = the batch's coefficient count); the cotangents of (xi, lambda, xi_bar) are carried
// between launches in `carry` ([3][stride]).
struct AdjFastArgs {
  const DevCfg* cfgs;
  const float* tab;
  const void* a32;               // basis operand tables of the MFMA kernels
  const DevProblem* probs;
  const WorkItem* items;
  int32_t n_items;
  const float* states;
  int64_t stride;
  int32_t every, seg0;           // checkpoint interval, first segment in `states`
  int32_t k_begin, k_end, iters; // the launch walks iterations k_end - 1 .. k_begin of iters
  const float* w_fpr;
  const float* g_resid;          // final-residual term only
  const float* g_xi_out;         // without the final-residual term the first launch starts from these
  const float* g_lam_out;
  bool init;                     // initialise the carries from g_xi_out / g_lam_out (else read them)
  float* carry;
  const float* pend;             // cotangent of xi^{K-1} from the final-residual term, or NULL
  float* pend_out;               // ... and where that term writes it
  float* g_xi0;                  // last launch (k_begin = 0): outputs instead of carries (any may be NULL)
  float* g_lam0;
  float* g_xi_bar;
  bool last;
  hipStream_t stream;
};

// Whether a config is covered by the MFMA adjoint path; the reverse sweep over the segments in `states`; the
// final-residual term (from the last two states, into the carries and pend_out).  R, KS: robot tiles of 16
// and coefficient steps of 4 of the whole batch, cfgs the configs it uses.
bool adjoint_fast_supported(const DevCfg& c);
hipError_t launch_adjoint_fast(const AdjFastArgs& a, const DevCfg* const* cfgs, int n_cfgs, int R, int KS, int ncu);
hipError_t launch_adjoint_resid(const AdjFastArgs& a, const DevCfg* const* cfgs, int n_cfgs, int R, int KS);

}  // namespace sf
