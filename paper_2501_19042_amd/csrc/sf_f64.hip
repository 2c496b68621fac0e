// FP64 solve on the matrix cores (2D and 3D, up to 32 robots, degree <= 15, horizon <= 256).
//
// One workgroup of W waves owns one sample; wave w owns the 16-step time tiles w, w + W, ...  An
// iteration has three barriers:
//   tiles (each wave): S1 as v_mfma_f64_16x16x4f64 (rows = 16 times, columns = 16 robots of one axis),
//     ball and workspace residuals in the product registers, pair residuals scattered into an LDS
//     accumulator, S4 as the same product with the rho-scaled basis, only for tiles with a nonzero
//     residual;
//   barrier; multiplier step and QP right-hand side y, one lane per (axis, free coefficient, robot), so
//     that the mean of y over the robots is a sum over aligned groups of 16R lanes;
//   barrier; QP step; barrier.
// Work whose result is exactly zero is skipped as in the fp32 kernels, by the same bounds: pairs whose
// position boxes over a tile are farther apart than the safety distance (lists kept until a robot may have
// moved by the margin), ball and workspace rows while a drift bound proves them inactive.  The tests are
// written so that a NaN lists the pair and evaluates the rows: a sample with NaN inputs goes through the
// dense kernel's arithmetic.
//
// What bounds it: the dependent chain of one iteration (about 11,000 cycles with one time tile per wave: the
// products 1,700, a v_mfma_f64_16x16x4f64 takes 64 cycles; pair and box tests 2,500; multiplier and QP
// steps 3,000; barriers 1,000), not the FP64 rate.  16 robots x 64 samples: 5.1 us per iteration, against
// 139 us in the dense generic kernel, which reads the basis from global memory for every product and takes
// a root and a division for every pair and time; 4 robots in 2D x 8 samples: 4.8 us against 34.6 us.
#include "sf_f64.h"

#include <algorithm>
#include <cfloat>
#include <cmath>

namespace sf {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma64(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)u, CTRL, 0xF, 0xF, false);
  const uint32_t hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(u >> 32), CTRL, 0xF, 0xF, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Sum over aligned groups of NR (16 or 32) lanes; every lane of a group gets the same value.
template <int NR>
__device__ __forceinline__ double group_sum(double v) {
  v = v + dpp<0xB1>(v);
  v = v + dpp<0x4E>(v);
  v = v + dpp<0x141>(v);
  v = v + dpp<0x140>(v);
  if constexpr (NR == 32) v = v + __shfl_xor(v, 16);
  return v;
}

// Maximum that keeps a NaN.
__device__ __forceinline__ double nan_max(double a, double b) { return (b > a || b != b) ? b : a; }

// LDS plan (in doubles; the pair table and lists are 16-bit).
struct F64Lds {
  int xi, lam, xb, y, ybar, xp, dx, x1, mx, red, pairs, tiles, per_wave, total;
  int xt, ct, bb, list;   // inside one wave's region
};

constexpr size_t kLds = 160 * 1024;
constexpr int kRows = 3;   // velocity, acceleration, workspace rows

__host__ __device__ inline F64Lds f64_plan(const DevCfg& c, int R, int W) {
  const int NR = 16 * R, D = c.D, nDm = c.n * D * c.m, nDf = c.n * D * c.mf, nD6 = c.n * D * kNFix;
  const int Np = c.n * (c.n - 1) / 2, TQ = ((c.H + 15) / 16 + W - 1) / W;
  F64Lds p;
  int o = 0;
  p.xi = o; o += nDm;
  p.lam = o; o += nDm;
  p.xb = o; o += nDm;
  p.y = o; o += nDf;                        // y; before the first step its correction
  p.ybar = o; o += D * c.mf;
  p.xp = o; o += nD6;                       // pinned coefficients (from the boundary values)
  p.x1 = o; o += 2 * c.mf * c.mf;           // X1, X01
  p.dx = o; o += D * NR / 2;                // fp32: largest change of a row's coefficients in the last step
  p.mx = o; o += kRows * NR;                // fp32 [2][kind][robot]: largest squares of the evaluated rows
  p.red = o; o += 3 * W;
  p.pairs = o; o += (Np + 3) / 4;           // i | j << 8
  p.tiles = o;
  p.xt = 0;                                 // positions, later the wave's partial back-projection
  p.ct = D * NR * 16;                       // residual accumulator, zero between tiles
  p.bb = 2 * D * NR * 16;                   // boxes: lo, hi per (axis, robot)
  p.list = p.bb + 2 * D * NR;               // per tile of the wave: count, then pair codes
  p.per_wave = p.list + (TQ * (Np + 1) + 3) / 4;
  o += W * p.per_wave;
  p.total = o;
  return p;
}

// (row, t) of a tile buffer, row = axis * 16R + robot: the 16 times of a row are rotated by the row, so
// that the 16 rows of one lane group fall in distinct banks.
__device__ __forceinline__ int at(int row, int t) { return row * 16 + ((t + row) & 15); }

struct F64Args {
  const DevCfg* cfgs;
  const double* tab;
  const double* a64;
  const DevProblem* probs;
  const WorkItem* items;
  int n_items;
  const double* xi_bar;
  const double* bvals;
  const double* xi0;
  const double* lam0;
  int iters;
  double* xi_out;
  double* lam_out;
  double* resid_out;
  int32_t* status_out;
  double* ckpt;
  int ckpt_every;
  int64_t ckpt_stride;
  int fpr;
};

// Residual of a pair (lower, upper) with separation r (alpha/beta/d steps in radial form).
template <int D>
__device__ __forceinline__ void pair_resid(const double (&r)[D], double ia2, double ib2, double a, double b,
                                           double (&o)[D]) {
  double ss = r[0] * r[0] * ia2 + r[1] * r[1] * ia2;
  if constexpr (D == 3) ss += r[2] * r[2] * ib2;
#pragma unroll
  for (int d = 0; d < D; ++d) o[d] = 0.0;
  if (ss >= DBL_MIN) {
    if (ss < 1.0) {   // farther apart: 1 - 1/||s|| >= 0 and the residual is zero
      const double f = fmin(0.0, 1.0 - 1.0 / sqrt(ss));
#pragma unroll
      for (int d = 0; d < D; ++d) o[d] = f * r[d];
    }
  } else if constexpr (D == 3) {   // coincident (or NaN): atan2(0, 0) = 0 targets (0, 0, b), (a, 0) in 2D
    o[2] = -b;
  } else {
    o[0] = -a;
  }
}

// (one robot tile: 256 registers, so that two samples of four waves, or one of eight, fit a CU)
template <int D, int R, int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(R == 1 ? 2 : 1, R == 1 ? 2 : 1)))
f64_project_kernel(F64Args A) {
  extern __shared__ __align__(16) double sm[];
  constexpr int NR = 16 * R, nthr = 64 * W;
  constexpr int NFI = (D * 10 * NR + nthr - 1) / nthr;       // free items per thread (degree <= 15)
  constexpr int NPI = (D * kNFix * NR + nthr - 1) / nthr;    // pinned items per thread
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tid = threadIdx.x, lane = tid & 63;
  const bool fpr = A.fpr != 0;
  const int rw = fpr ? 3 : 2;
  for (int it = blockIdx.x; it < A.n_items; it += gridDim.x) {
    const WorkItem w = A.items[it];
    const DevProblem pr = A.probs[w.problem];
    const DevCfg& c = A.cfgs[pr.cfg];
    const F64Lds L = f64_plan(c, R, W);
    const int n = c.n, m = c.m, mf = c.mf, H = c.H, nDm = n * D * m, nDf = n * D * mf, nD6 = n * D * kNFix;
    const int Np = n * (n - 1) / 2, NT = (H + 15) / 16, TQ = (NT + W - 1) / W, ks = (m + 3) / 4;
    const double *Bmap = A.tab + c.off_Bmap, *Gfx = A.tab + c.off_Gfx, *Rfx = A.tab + c.off_Rfx;
    const double ia2 = c.inv_a2, ib2 = c.inv_b2, sa = c.a, sb = c.b, vmax = c.vmax, amax = c.amax;
    const double inv_n = 1.0 / n, n_rho_c = c.n_rho_c, wsc = c.ws_scale;
    const double wc[3] = {c.ws_c[0], c.ws_c[1], c.ws_c[2]}, wi[3] = {c.ws_ia2, c.ws_ia2, c.ws_ib2};
    const bool vel_on = c.vel_on, acc_on = c.acc_on, ws_on = c.ws_on;
    const double skx = c.skin * c.a, skz = c.skin * c.b;
    const float fskx = 0.999f * (float)skx, fskz = 0.999f * (float)skz, fvmax = (float)vmax, famax = (float)amax;
    const float fLv = (float)c.lip_v, fLa = (float)c.lip_a, fwi[3] = {c.ws_f[3], c.ws_f[3], c.ws_f[4]};
    const d4* tabA = reinterpret_cast<const d4*>(A.a64 + c.off_a64);   // [tile][basis][S1, S4][lane]
    const double* bv = A.bvals + pr.bnd_off;
    double *sxi = sm + L.xi, *slam = sm + L.lam, *sxb = sm + L.xb, *sy = sm + L.y, *scorr = sy;
    double *sybar = sm + L.ybar, *sxp = sm + L.xp, *sX1 = sm + L.x1, *sX01 = sX1 + mf * mf;
    // bookkeeping of the drift bounds in fp32, as bits: non-negative floats order like their bits and a NaN
    // lies above all of them, so an integer maximum keeps it
    uint32_t* sdx = reinterpret_cast<uint32_t*>(sm + L.dx);   // [axis][robot]
    uint32_t* smx = reinterpret_cast<uint32_t*>(sm + L.mx);   // [iteration & 1][rows kind][robot]
    uint16_t* spairs = reinterpret_cast<uint16_t*>(sm + L.pairs);
    double* wbuf = sm + L.tiles + wave * L.per_wave;
    double *Xt = wbuf + L.xt, *Ct = wbuf + L.ct, *bb = wbuf + L.bb;
    uint16_t* lists = reinterpret_cast<uint16_t*>(wbuf + L.list);
    for (int q = tid; q < n * n; q += nthr) {
      const int i = q / n, j = q - i * n;
      if (j > i) spairs[i * n - i * (i + 1) / 2 + j - i - 1] = (uint16_t)(i | (j << 8));
    }
    for (int q = tid; q < mf * mf; q += nthr) {
      sX1[q] = (A.tab + c.off_X1)[q];
      sX01[q] = (A.tab + c.off_X01)[q];
    }
    // items of the multiplier and QP steps: (axis, free coefficient, robot) and (axis, pinned one, robot)
    // with the robot fastest; -1: none.  The pinned items start where the free ones end.
    int fi[NFI], fg[NFI], frow[NFI], ff[NFI], pi_[NPI], pg[NPI], pr6[NPI];
    // word of coefficient (robot, axis, kk) in a wave's partial back-projection, stored as the products leave
    // it: [axis][robot tile][r][lane], lane (col, grp) = (kk, robot of 4 r + grp)
    auto part_at = [](int robot, int d, int kk) {
      return ((d * R + (robot >> 4)) * 4 + ((robot & 15) >> 2)) * 64 + (robot & 3) * 16 + kk;
    };
    const int nfree = D * mf * NR, npin = D * kNFix * NR, rot = ((nfree + 63) & ~63) % nthr;
#pragma unroll
    for (int j = 0; j < NFI; ++j) {
      const int t = tid + j * nthr, rb = t % NR, f = mf > 0 ? (t / NR) % mf : 0, d = mf > 0 ? t / (NR * mf) : 0;
      const bool ok = t < nfree && rb < n;
      frow[j] = (ok ? rb * D : 0) + (t < nfree ? d : 0);
      ff[j] = t < nfree ? f : 0;
      fi[j] = ok ? frow[j] * m + 3 + f : -1;
      fg[j] = part_at(rb, t < nfree ? d : 0, 3 + f);
    }
#pragma unroll
    for (int j = 0; j < NPI; ++j) {
      const int t = (tid - rot + nthr) % nthr + j * nthr, rb = t % NR, r = (t / NR) % kNFix, d = t / (NR * kNFix);
      const bool ok = t < npin && rb < n;
      const int row = rb * D + d;
      pi_[j] = ok ? row * m + (r < 3 ? r : m - kNFix + r) : -1;
      pg[j] = ok ? part_at(rb, d, r < 3 ? r : m - kNFix + r) : 0;
      pr6[j] = ok ? row * kNFix + r : 0;
    }
    for (int sl = w.first; sl < w.first + w.count; ++sl) {
      const int64_t coef = pr.coef_off + (int64_t)sl * nDm;
      const int64_t sidx = pr.sample_base + sl;
      for (int q = tid; q < nDm; q += nthr) {
        const double x = A.xi_bar[coef + q];
        sxb[q] = x;
        sxi[q] = A.xi0 ? A.xi0[coef + q] : x;
        slam[q] = A.lam0 ? A.lam0[coef + q] : 0.0;
      }
      for (int q = tid; q < nD6; q += nthr) {
        const int row = q / kNFix, r = q - row * kNFix;
        double acc = 0.0;
        for (int s = 0; s < kNFix; ++s) acc = fma(Bmap[r * kNFix + s], bv[row * kNFix + s], acc);
        sxp[q] = acc;
      }
      const int32_t in_flag = A.status_out ? __builtin_amdgcn_readfirstlane(A.status_out[sidx]) : 0;
      const int iters = in_flag < 0 ? 0 : A.iters;   // (flagged by the input check: not iterated)
      __syncthreads();
      // first-step correction G_rho (xi0 - xi_p) on the free coefficients (its operands in the first
      // wave's tile region)
      double *sdl = sm + L.tiles, *sdb = sdl + nD6;
      for (int q = tid; q < nD6; q += nthr) {
        const int row = q / kNFix, r = q - row * kNFix;
        sdl[q] = sxi[row * m + (r < 3 ? r : m - kNFix + r)] - sxp[q];
      }
      __syncthreads();
      for (int q = tid; q < D * kNFix; q += nthr) {
        const int d = q / kNFix, r = q - d * kNFix;
        double s = 0.0;
        for (int i = 0; i < n; ++i) s += sdl[(i * D + d) * kNFix + r];
        sdb[q] = s * inv_n;
      }
      __syncthreads();
      for (int q = tid; q < nDf; q += nthr) {
        const int row = q / mf, f = q - row * mf, d = row % D;
        double acc = 0.0;
        for (int r = 0; r < kNFix; ++r) {
          const double dl = sdl[row * kNFix + r];
          acc = fma(n_rho_c * Gfx[f * kNFix + r], dl - sdb[d * kNFix + r], acc);
          acc = fma(Rfx[f * kNFix + r], dl, acc);
        }
        scorr[q] = acc;
      }
      __syncthreads();
      for (int q = lane; q < D * NR * 16; q += 64) Ct[q] = 0.0;
      // position operands of the wave's first tile, held for all iterations
      d4 p0a = {0.0, 0.0, 0.0, 0.0}, p0b = {0.0, 0.0, 0.0, 0.0};
      if (wave < NT) {
        p0a = tabA[((wave * 3) * 2) * 64 + lane];
        p0b = tabA[((wave * 3) * 2 + 1) * 64 + lane];
      }
      // per robot (lane), identical in every wave: slack to the velocity, acceleration and workspace
      // bounds at the last evaluation less the drift since, and drift since the pair lists were built
      float sv = -1.0f, sacc = -1.0f, sws = -1.0f, px[D];
#pragma unroll
      for (int d = 0; d < D; ++d) px[d] = 0.0f;
      for (int q = tid; q < D * NR; q += nthr) sdx[q] = 0u;
      for (int q = tid; q < 2 * kRows * NR; q += nthr) smx[q] = 0u;
      int prev_eval = 0;
      double fsum = 0.0;
      __syncthreads();
      for (int k = 0; k < iters; ++k) {
        // per-lane indices from an opaque copy, so that the compiler does not hoist every per-lane
        // address of the loop body out of the loop and spill it
        int tid_k = threadIdx.x;
        asm volatile("" : "+v"(tid_k));
        const int tid = tid_k, lane = tid_k & 63, col = lane & 15, grp = lane >> 4;
        if (A.ckpt && (k % A.ckpt_every) == 0) {
          const int64_t base = (int64_t)(k / A.ckpt_every) * 2 * A.ckpt_stride + coef;
          for (int q = tid; q < nDm; q += nthr) {
            A.ckpt[base + q] = sxi[q];
            A.ckpt[base + A.ckpt_stride + q] = slam[q];
          }
        }
        if ((A.resid_out || A.status_out) && k == iters - 1)
          for (int q = tid; q < nDm; q += nthr) A.xi_out[coef + q] = sxi[q];   // overwritten with the result
        // What to evaluate: a position, velocity or acceleration moves per step by at most its basis'
        // largest row sum times the largest change of a coefficient.
        int eval = 7;
        bool rebuild = true;
        {
          bool ev = false, ea = false, ew = false, er = false;
          if (lane < n) {
            // (hardware square roots: the tests keep a 1e-4 relative slack, far above the fp32 rounding)
            const uint32_t* pm = smx + ((k + 1) & 1) * kRows * NR + lane;
            auto worst = [&](int kind) { return __builtin_amdgcn_sqrtf(__uint_as_float(pm[kind * NR])); };
            if (prev_eval & 1) sv = fvmax - worst(0);
            if (prev_eval & 2) sacc = famax - worst(1);
            if (prev_eval & 4) sws = 1.0f - worst(2);
            float dn = 0.0f, dw = 0.0f;
#pragma unroll
            for (int d = 0; d < D; ++d) {
              const float mx = __uint_as_float(sdx[d * NR + lane]);
              px[d] = drift_add(px[d], mx);
              dn = fmaf(mx, mx, dn);
              dw = fmaf(mx * mx, fwi[d], dw);
              er |= !(px[d] <= (d == 2 ? fskz : fskx));
            }
            dn = __builtin_amdgcn_sqrtf(dn) + 2e-19f;   // (squares below the smallest float vanish)
            sv = slack_less(sv, fLv * dn);
            sacc = slack_less(sacc, fLa * dn);
            if (ws_on) sws = slack_less(sws, __builtin_amdgcn_sqrtf(dw));
            ev = !(sv > 1e-4f * fvmax);
            ea = !(sacc > 1e-4f * famax);
            ew = !(sws > 1e-4f);
          }
          if (k >= 2) {
            eval = (__ballot(ev) ? 1 : 0) | (__ballot(ea) ? 2 : 0) | (__ballot(ew) ? 4 : 0);
            rebuild = __ballot(er) != 0;
          }
          eval &= (vel_on ? 1 : 0) | (acc_on ? 2 : 0) | (ws_on ? 4 : 0);
          prev_eval = eval;
        }
        double mg[D];
        if (rebuild) {
          // margins of the broad phase: twice the drift margin plus the rounding of a position (a convex
          // combination of at most 16 coefficients: 1e-14 of the largest)
          double cm = 0.0;
          for (int q = lane; q < nDm; q += 64) cm = fmax(cm, fabs(sxi[q]));
          if (k == 0)   // (later ones are in xi)
            for (int q = lane; q < nD6; q += 64) cm = fmax(cm, fabs(sxp[q]));
          for (int off = 32; off > 0; off >>= 1) cm = fmax(cm, __shfl_xor(cm, off));
          const double tol = 1e-10 * (cm + fmax(skx, skz));
#pragma unroll
          for (int d = 0; d < D; ++d) {
            px[d] = 0.0f;
            mg[d] = 2.0 * (d == 2 ? skz : skx) + tol;
          }
        }
        // S1 B operand: lane (col, grp) holds robot col, coefficient 4 s + grp
        double bx[R][D][4];
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
          for (int d = 0; d < D; ++d)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
              const int robot = 16 * rr + col, kk = 4 * s + grp;
              bx[rr][d][s] = (robot < n && kk < m) ? sxi[(robot * D + d) * m + kk] : 0.0;
            }
        // Y[rr][d][r]: robot 16 rr + col at time 4 r + grp of the tile
        auto s1 = [&](const d4 a, d4 (&Y)[R][D]) {
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int d = 0; d < D; ++d) Y[rr][d] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int s = 0; s < 4; ++s)
            if (s < ks) {
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int d = 0; d < D; ++d) Y[rr][d] = mfma64(a[s], bx[rr][d][s], Y[rr][d]);
            }
        };
        d4 g[R][D];
        double vm[kRows][R];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
#pragma unroll
          for (int d = 0; d < D; ++d) g[rr][d] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
          for (int b = 0; b < kRows; ++b) vm[b][rr] = 0.0;
        }
#pragma unroll 1
        for (int q = 0; q < TQ; ++q) {
          const int tau = wave + W * q;
          if (tau >= NT) break;
          const int nt = min(16, H - 16 * tau);
          uint16_t* tl = lists + q * (Np + 1);
          int count = rebuild ? 0 : (int)tl[0];
          bool wnz = false;
          if (rebuild || count > 0 || (eval & 4)) {
            d4 Y[R][D];
            s1(q == 0 ? p0a : tabA[((tau * 3) * 2) * 64 + lane], Y);
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < D; ++d)
#pragma unroll
                for (int r = 0; r < 4; ++r) Xt[at(d * NR + 16 * rr + col, 4 * r + grp)] = Y[rr][d][r];
            if (eval & 4) {
              // workspace rows on the same positions, scaled by rho_w / rho_c so that they share the
              // collision residuals' accumulator
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  double qd[D], ss = 0.0;
#pragma unroll
                  for (int d = 0; d < D; ++d) {
                    qd[d] = Y[rr][d][r] - wc[d];
                    ss += qd[d] * qd[d] * wi[d];
                  }
                  const bool real = 16 * rr + col < n;
                  vm[2][rr] = nan_max(vm[2][rr], ss);
                  const double f = ss > 1.0 ? 1.0 - 1.0 / sqrt(ss) : 0.0;
#pragma unroll
                  for (int d = 0; d < D; ++d) {
                    const double v = real ? wsc * (f * qd[d]) : 0.0;
                    Y[rr][d][r] = v;
                    wnz |= v != 0.0;
                  }
                }
              wnz = __ballot(wnz) != 0;
              if (wnz) {
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int d = 0; d < D; ++d)
#pragma unroll
                    for (int r = 0; r < 4; ++r) Ct[at(d * NR + 16 * rr + col, 4 * r + grp)] = Y[rr][d][r];
              }
            }
          }
#pragma unroll
          for (int b = 1; b < 3; ++b) {
            if (!(eval & b)) continue;
            const double lim = b == 1 ? vmax : amax;
            d4 Y[R][D];
            s1(tabA[((tau * 3 + b) * 2) * 64 + lane], Y);
            bool out = false;
            double ss[R][4];
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                double v = Y[rr][0][r] * Y[rr][0][r] + Y[rr][1][r] * Y[rr][1][r];
                if constexpr (D == 3) v += Y[rr][2][r] * Y[rr][2][r];
                ss[rr][r] = v;
                vm[b - 1][rr] = nan_max(vm[b - 1][rr], v);
                out |= !(v <= lim * lim);
              }
            if (__ballot(out) == 0) continue;
            bool nz = false;
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const double f = ss[rr][r] > lim * lim ? 1.0 - lim * (1.0 / sqrt(ss[rr][r])) : 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                  Y[rr][d][r] = f * Y[rr][d][r];
                  nz |= Y[rr][d][r] != 0.0;
                }
              }
            if (__ballot(nz) != 0) {
              const d4 bq = tabA[((tau * 3 + b) * 2 + 1) * 64 + lane];
#pragma unroll
              for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int d = 0; d < D; ++d) g[rr][d] = mfma64(Y[rr][d][s], bq[s], g[rr][d]);
            }
          }
          wave_sync();
          if (rebuild) {
            for (int row = lane; row < D * NR; row += 64) {
              double lo = Xt[at(row, 0)], hi = lo;
#pragma unroll
              for (int t = 1; t < 16; ++t) {   // (rows past the horizon repeat the last grid time)
                const double v = Xt[at(row, t)];
                lo = fmin(lo, v);
                hi = fmax(hi, v);
              }
              bb[2 * row] = lo;
              bb[2 * row + 1] = hi;
            }
            wave_sync();
            for (int base = 0; base < Np; base += 64) {
              const int p = base + lane;
              const int code = spairs[min(p, Np - 1)], i = code & 255, j = code >> 8;
              double g2 = 0.0;
#pragma unroll
              for (int d = 0; d < D; ++d) {
                const double* bi = bb + 2 * (d * NR + i);
                const double* bj = bb + 2 * (d * NR + j);
                double gap = nan_max(bj[0] - bi[1], bi[0] - bj[1]) - mg[d];
                gap = gap < 0.0 ? 0.0 : gap;   // (a NaN box stays NaN and its pairs are listed)
                g2 += gap * gap * (d == 2 ? ib2 : ia2);
              }
              const bool act = p < Np && !(g2 >= 1.000001);
              const uint64_t mask = __ballot(act);
              if (act)
                tl[1 + count + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                         __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0))] = (uint16_t)code;
              count += __popcll(mask);
            }
            if (lane == 0) tl[0] = (uint16_t)count;
            wave_sync();
          }
          count = __builtin_amdgcn_readfirstlane(count);
          const int tsh = nt <= 4 ? 2 : (nt <= 8 ? 3 : 4);
          const int tt = lane & ((1 << tsh) - 1), ps = lane >> tsh, ppr = 64 >> tsh;
          bool nzc = false;
          for (int base = 0; base < count; base += ppr) {
            const int slot = base + ps;
            if (slot < count && tt < nt) {
              const int code = tl[1 + slot], i = code & 255, j = code >> 8;
              double r[D], o[D];
              bool nz = false;
#pragma unroll
              for (int d = 0; d < D; ++d) r[d] = Xt[at(d * NR + i, tt)] - Xt[at(d * NR + j, tt)];
              pair_resid<D>(r, ia2, ib2, sa, sb, o);
#pragma unroll
              for (int d = 0; d < D; ++d) nz |= o[d] != 0.0;
              if (nz) {
                nzc = true;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                  atomicAdd(Ct + at(d * NR + i, tt), o[d]);
                  atomicAdd(Ct + at(d * NR + j, tt), -o[d]);
                }
              }
            }
          }
          if (wnz || __ballot(nzc) != 0) {
            wave_sync();
            const d4 cb = q == 0 ? p0b : tabA[((tau * 3) * 2 + 1) * 64 + lane];
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int d = 0; d < D; ++d) {
                  double* cp = Ct + at(d * NR + 16 * rr + col, 4 * s + grp);
                  const double v = *cp;
                  *cp = 0.0;
                  g[rr][d] = mfma64(v, cb[s], g[rr][d]);
                }
          }
          wave_sync();
        }
        // partial back-projection (lane (col, grp): coefficient col, robots 4 r + grp) and the maxima
#pragma unroll
        for (int d = 0; d < D; ++d)
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int r = 0; r < 4; ++r) Xt[((d * R + rr) * 4 + r) * 64 + lane] = g[rr][d][r];
#pragma unroll
        for (int b = 0; b < kRows; ++b)
          if (eval & (1 << b)) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
              atomicMax(smx + ((k & 1) * kRows + b) * NR + 16 * rr + col, __float_as_uint((float)vm[b][rr]));
          }
        __syncthreads();
        // multiplier step, and y = xi_bar - xi + lambda - g with its robot mean
        const double* part = sm + L.tiles;
        auto gsum = [&](int q) {
          double s = part[q];
#pragma unroll
          for (int ww = 1; ww < W; ++ww) s += part[ww * L.per_wave + q];
          return s;
        };
        for (int q = tid; q < D * NR; q += nthr) sdx[q] = 0u;
        for (int q = tid; q < kRows * NR; q += nthr) smx[((k + 1) & 1) * kRows * NR + q] = 0u;
#pragma unroll
        for (int j = 0; j < NFI; ++j) {
          if (tid - lane + j * nthr >= nfree) break;   // (uniform over the wave)
          const int q = fi[j];
          double y = 0.0;
          if (q >= 0) {
            const double gq = gsum(fg[j]), ln = slam[q] - gq;
            slam[q] = ln;
            y = sxb[q] - sxi[q] + ln - gq;
            if (k == 0) y += scorr[frow[j] * mf + ff[j]];
            if (fpr) fsum = fma(gq, gq, fsum);
            sy[frow[j] * mf + ff[j]] = y;
          }
          const double ym = group_sum<NR>(y) * inv_n;
          if (lane % NR == 0 && tid + j * nthr < nfree) sybar[(frow[j] % D) * mf + ff[j]] = ym;
        }
#pragma unroll
        for (int j = 0; j < NPI; ++j) {
          const int q = pi_[j];
          if (q >= 0) {
            const double gq = gsum(pg[j]);
            slam[q] -= gq;
            if (fpr) fsum = fma(gq, gq, fsum);
            if (k == 0) {   // the boundary values are set in the first step
              const double xp = sxp[pr6[j]], dx = xp - sxi[q];
              if (fpr) fsum = fma(dx, dx, fsum);
              sxi[q] = xp;
            }
          }
        }
        __syncthreads();
        // QP step: xi_free += X1 y + X01 mean(y)
#pragma unroll
        for (int j = 0; j < NFI; ++j) {
          const int q = fi[j];
          if (q >= 0) {
            const int row = frow[j], f = ff[j], d = row % D;
            double acc = 0.0;
#pragma unroll 5
            for (int f2 = 0; f2 < mf; ++f2) {
              acc = fma(sX1[f * mf + f2], sy[row * mf + f2], acc);
              acc = fma(sX01[f * mf + f2], sybar[d * mf + f2], acc);
            }
            sxi[q] += acc;
            atomicMax(sdx + d * NR + row / D, __float_as_uint((float)fabs(acc)));
            if (fpr) fsum = fma(acc, acc, fsum);
          }
        }
        __syncthreads();
      }

      // ---- primal residual of the last step, dense over pairs ----
      int tid_r = threadIdx.x;
      asm volatile("" : "+v"(tid_r));
      const int tid = tid_r, lane = tid_r & 63, col = lane & 15, grp = lane >> 4;
      double rmax = 0.0;
      if (A.resid_out || A.status_out) {
        double ss = 0.0, mx = 0.0;
        if (iters > 0) {
          auto prod = [&](const double* src, int tau, int b, d4 (&Y)[R][D]) {
            const d4 a = tabA[((tau * 3 + b) * 2) * 64 + lane];
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < D; ++d) {
                Y[rr][d] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                  const int robot = 16 * rr + col, kk = 4 * s + grp;
                  const double v = (robot < n && kk < m) ? src[(robot * D + d) * m + kk] : 0.0;
                  if (s < ks) Y[rr][d] = mfma64(a[s], v, Y[rr][d]);
                }
              }
          };
          auto add = [&](const double (&rp)[D], bool real) {
            double nrm = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) nrm += rp[d] * rp[d];
            if (real) {
              ss += nrm;
              mx = nan_max(mx, nrm);
            }
          };
#pragma unroll 1
          for (int q = 0; q < TQ; ++q) {
            const int tau = wave + W * q;
            if (tau >= NT) break;
            const int nt = min(16, H - 16 * tau);
#pragma unroll 1
            for (int b = 0; b < 3; ++b) {
              if (b > 0 && !(b == 1 ? vel_on : acc_on)) continue;
              const double lim = b == 1 ? vmax : amax;
              d4 Y[R][D], Z[R][D];
              prod(A.xi_out + coef, tau, b, Y);
              prod(sxi, tau, b, Z);
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const bool real = 16 * rr + col < n && 4 * r + grp < nt;
                  double rp[D], s2 = 0.0;
                  if (b == 0) {
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                      Xt[at(d * NR + 16 * rr + col, 4 * r + grp)] = Y[rr][d][r];
                      Ct[at(d * NR + 16 * rr + col, 4 * r + grp)] = Z[rr][d][r];
                      const double v = Y[rr][d][r] - wc[d];
                      s2 += v * v * wi[d];
                    }
                    if (ws_on) {
                      const double f = s2 > 1.0 ? 1.0 - 1.0 / sqrt(s2) : 0.0;
#pragma unroll
                      for (int d = 0; d < D; ++d) rp[d] = Z[rr][d][r] - (Y[rr][d][r] - f * (Y[rr][d][r] - wc[d]));
                      add(rp, real);
                    }
                  } else {
#pragma unroll
                    for (int d = 0; d < D; ++d) s2 += Y[rr][d][r] * Y[rr][d][r];
                    const double f = s2 > lim * lim ? 1.0 - lim * (1.0 / sqrt(s2)) : 0.0;
#pragma unroll
                    for (int d = 0; d < D; ++d) rp[d] = Z[rr][d][r] - (Y[rr][d][r] - f * Y[rr][d][r]);
                    add(rp, real);
                  }
                }
            }
            wave_sync();
            const int tsh = nt <= 4 ? 2 : (nt <= 8 ? 3 : 4);
            const int tt = lane & ((1 << tsh) - 1), ps = lane >> tsh, ppr = 64 >> tsh;
            for (int slot = ps; slot < Np; slot += ppr)
              if (tt < nt) {
                const int code = spairs[slot], i = code & 255, j = code >> 8;
                double r[D], o[D], rp[D];
#pragma unroll
                for (int d = 0; d < D; ++d) r[d] = Xt[at(d * NR + i, tt)] - Xt[at(d * NR + j, tt)];
                pair_resid<D>(r, ia2, ib2, sa, sb, o);
#pragma unroll
                for (int d = 0; d < D; ++d)
                  rp[d] = (Ct[at(d * NR + i, tt)] - Ct[at(d * NR + j, tt)]) - (r[d] - o[d]);
                add(rp, true);
              }
            wave_sync();
          }
        }
        for (int off = 32; off > 0; off >>= 1) {
          ss += __shfl_xor(ss, off);
          mx = nan_max(mx, __shfl_xor(mx, off));
          fsum += __shfl_xor(fsum, off);
        }
        double* red = sm + L.red;
        if (lane == 0) {
          red[3 * wave] = ss;
          red[3 * wave + 1] = mx;
          red[3 * wave + 2] = fsum;
        }
        __syncthreads();
        if (tid == 0) {
          double s = 0.0, mm = 0.0, fs = 0.0;
          for (int ww = 0; ww < W; ++ww) {
            s += red[3 * ww];
            mm = nan_max(mm, red[3 * ww + 1]);
            fs += red[3 * ww + 2];
          }
          rmax = sqrt(mm);
          if (A.resid_out) {
            A.resid_out[sidx * rw] = s;
            A.resid_out[sidx * rw + 1] = rmax;
            if (fpr) A.resid_out[sidx * rw + 2] = fs;
          }
        }
        __syncthreads();
      }
      for (int q = tid; q < nDm; q += nthr) {
        A.xi_out[coef + q] = sxi[q];
        if (A.lam_out) A.lam_out[coef + q] = slam[q];
      }
      if (A.status_out && tid == 0)
        A.status_out[sidx] = in_flag < 0 ? in_flag : sample_status<double>(false, false, rmax, iters);
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------------------------
// FP64 feasibility check at the grid times, four waves per sample, time tiles as above.  The largest speeds
// and workspace offsets come from the product registers.  The smallest separation of a tile is first taken at
// one of its times; then only pairs whose boxes are nearer than that are visited at all of them, so the
// minimum is that over every pair and time.  Bound by the FP64 matrix rate (16 robots: 27 products a tile of
// 64 cycles, 5 us at 1024 samples) and the LDS reads of the pairs: 26 us, against 97 us in the generic kernel,
// which visits every pair at every time and reads the basis from global memory.
// ---------------------------------------------------------------------------------

constexpr int kCheckW = 4;

struct CheckLds {
  int x, red, pairs, tiles, per_wave, total;   // in doubles
  int xt, bb, list;
};

__host__ __device__ inline CheckLds check_plan(const DevCfg& c, int R) {
  const int NR = 16 * R, D = c.D, Np = c.n * (c.n - 1) / 2;
  CheckLds p;
  int o = 0;
  p.x = o; o += D * 16 * NR;                // [axis][16 coefficients][16R robots], zero outside
  p.red = o; o += 5 * kCheckW;
  p.pairs = o; o += (Np + 3) / 4;
  p.tiles = o;
  p.xt = 0;
  p.bb = D * NR * 16;
  p.list = p.bb + 2 * D * NR;
  p.per_wave = p.list + (Np + 3) / 4;
  o += kCheckW * p.per_wave;
  p.total = o;
  return p;
}

template <typename Tin, int D, int R>
__global__ void __launch_bounds__(64 * kCheckW)
f64_check_kernel(const DevCfg* __restrict__ cfgs, const double* __restrict__ tab, const double* __restrict__ a64,
                 const DevProblem* __restrict__ probs, const WorkItem* __restrict__ items, int n_items,
                 const Tin* __restrict__ xi, const Tin* __restrict__ bvals, double* __restrict__ viol) {
  extern __shared__ __align__(16) double sm[];
  constexpr int NR = 16 * R, nthr = 64 * kCheckW;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, grp = lane >> 4;
  for (int it = blockIdx.x; it < n_items; it += gridDim.x) {
    const WorkItem w = items[it];
    const DevProblem pr = probs[w.problem];
    const DevCfg& c = cfgs[pr.cfg];
    const CheckLds L = check_plan(c, R);
    const int n = c.n, m = c.m, H = c.H, nDm = n * D * m, Np = n * (n - 1) / 2, NT = (H + 15) / 16, ks = (m + 3) / 4;
    const double ia2 = c.inv_a2, ib2 = c.inv_b2;
    const double wc[3] = {c.ws_c[0], c.ws_c[1], c.ws_c[2]}, wi[3] = {c.ws_ia2, c.ws_ia2, c.ws_ib2};
    const double* basis = tab + c.off_basis;
    const d4* tabA = reinterpret_cast<const d4*>(a64 + c.off_a64);
    const Tin* bv = bvals + pr.bnd_off;
    double *x = sm + L.x, *red = sm + L.red, *wbuf = sm + L.tiles + wave * L.per_wave;
    double *Xt = wbuf + L.xt, *bb = wbuf + L.bb;
    uint16_t* spairs = reinterpret_cast<uint16_t*>(sm + L.pairs);
    uint16_t* tl = reinterpret_cast<uint16_t*>(wbuf + L.list);
    for (int q = tid; q < D * 16 * NR; q += nthr) x[q] = 0.0;
    for (int q = tid; q < n * n; q += nthr) {
      const int i = q / n, j = q - i * n;
      if (j > i) spairs[i * n - i * (i + 1) / 2 + j - i - 1] = (uint16_t)(i | (j << 8));
    }
    __syncthreads();
    for (int sl = w.first; sl < w.first + w.count; ++sl) {
      const int64_t coef = pr.coef_off + (int64_t)sl * nDm;
      const int64_t sidx = pr.sample_base + sl;
      for (int q = tid; q < nDm; q += nthr) {
        const int row = q / m, k = q - row * m, i = row / D, d = row - i * D;
        x[(d * 16 + k) * NR + i] = (double)xi[coef + q];
      }
      __syncthreads();
      double smin = DBL_MAX, vmx = 0.0, amx = 0.0, bmx = 0.0, wmx = 0.0;
      for (int q = tid; q < n * D * kNFix; q += nthr) {
        const int row = q / kNFix, r = q - row * kNFix, i = row / D, d = row - i * D;
        const double* brow = basis + ((size_t)(r % 3) * H + (r < 3 ? 0 : H - 1)) * m;
        double acc = 0.0;
#pragma unroll 4
        for (int k = 0; k < m; ++k) acc = fma(brow[k], x[(d * 16 + k) * NR + i], acc);
        bmx = fmax(bmx, fabs(acc - (double)bv[q]));
      }
      auto prod = [&](const d4 a, d4 (&Y)[R][D]) {
        const double* xp = x + grp * NR + col;
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
          for (int d = 0; d < D; ++d) Y[rr][d] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s)
          if (s < ks) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < D; ++d) Y[rr][d] = mfma64(a[s], xp[(d * 16 + 4 * s) * NR + 16 * rr], Y[rr][d]);
          }
      };
#pragma unroll 1
      for (int tau = wave; tau < NT; tau += kCheckW) {
        d4 Y[R][D];
        // (rows past the horizon repeat the last grid time: no other value enters)
        prod(tabA[(tau * 3 * 2) * 64 + lane], Y);
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double w2 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
              Xt[at(d * NR + 16 * rr + col, 4 * r + grp)] = Y[rr][d][r];
              const double v = Y[rr][d][r] - wc[d];
              w2 += v * v * wi[d];
            }
            if (16 * rr + col < n) wmx = fmax(wmx, w2);
          }
#pragma unroll 1
        for (int b = 1; b < 3; ++b) {
          prod(tabA[((tau * 3 + b) * 2) * 64 + lane], Y);
          double mx = 0.0;
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              double v2 = 0.0;
#pragma unroll
              for (int d = 0; d < D; ++d) v2 += Y[rr][d][r] * Y[rr][d][r];
              if (16 * rr + col < n) mx = fmax(mx, v2);
            }
          if (b == 1) vmx = fmax(vmx, mx);
          else amx = fmax(amx, mx);
        }
        wave_sync();
        for (int row = lane; row < D * NR; row += 64) {
          double lo = Xt[at(row, 0)], hi = lo;
#pragma unroll
          for (int t = 1; t < 16; ++t) {
            const double v = Xt[at(row, t)];
            lo = fmin(lo, v);
            hi = fmax(hi, v);
          }
          bb[2 * row] = lo;
          bb[2 * row + 1] = hi;
        }
        auto sep = [&](int code, int t) {
          const int i = code & 255, j = code >> 8;
          double s = 0.0;
#pragma unroll
          for (int d = 0; d < D; ++d) {
            const double r = Xt[at(d * NR + i, t)] - Xt[at(d * NR + j, t)];
            s += r * r * (d == 2 ? ib2 : ia2);
          }
          return s;
        };
        for (int p = lane; p < Np; p += 64) smin = fmin(smin, sep(spairs[p], 0));
        double near = smin;
        for (int off = 32; off > 0; off >>= 1) near = fmin(near, __shfl_xor(near, off));
        wave_sync();
        int count = 0;
        for (int base = 0; base < Np; base += 64) {
          const int p = base + lane;
          const int code = spairs[min(p, Np - 1)], i = code & 255, j = code >> 8;
          double g2 = 0.0;
#pragma unroll
          for (int d = 0; d < D; ++d) {
            const double* bi = bb + 2 * (d * NR + i);
            const double* bj = bb + 2 * (d * NR + j);
            const double gap = fmax(0.0, fmax(bj[0] - bi[1], bi[0] - bj[1]));
            g2 += gap * gap * (d == 2 ? ib2 : ia2);
          }
          const bool act = p < Np && g2 * (1.0 - 1e-12) < near;   // (far above the rounding of a gap)
          const uint64_t mask = __ballot(act);
          if (act)
            tl[count + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0))] = (uint16_t)code;
          count += __popcll(mask);
        }
        wave_sync();
        for (int slot = grp; slot < count; slot += 4) smin = fmin(smin, sep(tl[slot], col));
        wave_sync();
      }
      for (int off = 32; off > 0; off >>= 1) {
        smin = fmin(smin, __shfl_xor(smin, off));
        vmx = fmax(vmx, __shfl_xor(vmx, off));
        amx = fmax(amx, __shfl_xor(amx, off));
        bmx = fmax(bmx, __shfl_xor(bmx, off));
        wmx = fmax(wmx, __shfl_xor(wmx, off));
      }
      if (lane == 0) {
        double* rp = red + 5 * wave;
        rp[0] = smin;
        rp[1] = vmx;
        rp[2] = amx;
        rp[3] = bmx;
        rp[4] = wmx;
      }
      __syncthreads();
      if (tid == 0) {
        double v[5];
        for (int q = 0; q < 5; ++q) {
          v[q] = red[q];
          for (int ww = 1; ww < kCheckW; ++ww) v[q] = q == 0 ? fmin(v[q], red[5 * ww]) : fmax(v[q], red[5 * ww + q]);
        }
        viol[sidx * 5 + 0] = c.a * (1.0 - sqrt(v[0]));
        viol[sidx * 5 + 1] = c.vel_on ? sqrt(v[1]) - c.vmax : -DBL_MAX;
        viol[sidx * 5 + 2] = c.acc_on ? sqrt(v[2]) - c.amax : -DBL_MAX;
        viol[sidx * 5 + 3] = v[3];
        viol[sidx * 5 + 4] = c.ws_on ? c.ws_a * (sqrt(v[4]) - 1.0) : 0.0;
      }
      __syncthreads();
    }
  }
}

template <typename Tin, int D, int R>
hipError_t launch_check(const CheckArgs& a) {
  auto kern = f64_check_kernel<Tin, D, R>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)a.lds_bytes);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.n_items), dim3(64 * kCheckW), a.lds_bytes, a.stream, a.cfgs, a.tab, a.a64, a.probs,
                     a.items, a.n_items, static_cast<const Tin*>(a.xi), static_cast<const Tin*>(a.bvals), a.viol);
  return hipGetLastError();
}

template <int D, int R, int W>
hipError_t launch_instance(const F64Args& f, size_t lds, hipStream_t stream) {
  auto kern = f64_project_kernel<D, R, W>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(f.n_items), dim3(64 * W), lds, stream, f);
  return hipGetLastError();
}

}  // namespace

int64_t a64_entries(const DevCfg& c) { return (int64_t)((c.H + 15) / 16) * 3 * 2 * 64 * 4; }

void a64_fill(const DevCfg& c, const double* P3, double* out) {
  const int NT = (c.H + 15) / 16;
  const double rho[3] = {c.rho_c, c.rho_v, c.rho_a};
  for (int tau = 0; tau < NT; ++tau)
    for (int b = 0; b < 3; ++b)
      for (int lane = 0; lane < 64; ++lane) {
        const int col = lane & 15, grp = lane >> 4;
        // S1: P[t = 16 tau + col][k = 4 s + grp] (times past the horizon repeat the last grid time);
        // S4: rho P[t = 16 tau + 4 s + grp][k = col], zero past the horizon
        double* a = out + ((((size_t)tau * 3 + b) * 2 + 0) * 64 + lane) * 4;
        double* bq = out + ((((size_t)tau * 3 + b) * 2 + 1) * 64 + lane) * 4;
        for (int s = 0; s < 4; ++s) {
          const int t = std::min(16 * tau + col, c.H - 1), k = 4 * s + grp, t4 = 16 * tau + 4 * s + grp;
          a[s] = k < c.m ? P3[((size_t)b * c.H + t) * c.m + k] : 0.0;
          bq[s] = (t4 < c.H && col < c.m) ? rho[b] * P3[((size_t)b * c.H + t4) * c.m + col] : 0.0;
        }
      }
}

size_t f64_lds_bytes(const DevCfg& c, int R, int W) { return (size_t)f64_plan(c, R, W).total * sizeof(double); }

bool f64_cfg_covered(const DevCfg& c) {
  return c.n <= 32 && c.m <= 16 && c.H <= 256 && f64_lds_bytes(c, c.n <= 16 ? 1 : 2, c.n <= 16 ? 4 : 3) <= kLds;
}

// Whether the drift bounds can be kept in fp32: their squares must neither vanish nor overflow, so every length and
// rate of the config lies between 1e-9 and 1e9 of its units (in kilometres the workloads here have 1e-4, in
// millimetres 1e4).  Swarms outside, in units of 1e-22 m for instance, go through the kernel without such bounds.
static bool f64_units_covered(const DevCfg& c) {
  auto in = [](double v) { return v >= 1e-9 && v <= 1e9; };
  return in(c.a) && in(c.b) && (!c.vel_on || in(c.vmax)) && (!c.acc_on || in(c.amax)) &&
         (!c.ws_on || (in(c.ws_a) && in(1.0 / sqrt(c.ws_ib2))));
}

// Waves per sample: with one robot tile 8 while every sample has a CU of its own (one time tile per wave
// up to a horizon of 128), else 4, which keeps two samples per CU; with two robot tiles the LDS holds 4, or
// 3 at the largest polynomials.
int f64_waves(const DevCfg* const* cfgs, int n_cfgs, int R, int64_t n_items, int ncu, size_t* lds) {
  for (int i = 0; i < n_cfgs; ++i)
    if (!f64_units_covered(*cfgs[i])) return 0;
  for (int W : {8, 4, 3}) {
    if (W == 8 && (R == 2 || n_items > ncu)) continue;
    if (W == 3 && R == 1) continue;
    *lds = 0;
    for (int i = 0; i < n_cfgs; ++i) *lds = std::max(*lds, f64_lds_bytes(*cfgs[i], R, W));
    if (*lds <= kLds) return W;
  }
  return 0;
}

size_t f64_check_lds_bytes(const DevCfg& c, int R) { return (size_t)check_plan(c, R).total * sizeof(double); }

hipError_t launch_f64_check(const CheckArgs& a, bool dbl, int D, int R) {
  switch (D * 100 + R * 10 + (dbl ? 1 : 0)) {
    case 210: return launch_check<float, 2, 1>(a);
    case 211: return launch_check<double, 2, 1>(a);
    case 220: return launch_check<float, 2, 2>(a);
    case 221: return launch_check<double, 2, 2>(a);
    case 310: return launch_check<float, 3, 1>(a);
    case 311: return launch_check<double, 3, 1>(a);
    case 320: return launch_check<float, 3, 2>(a);
    case 321: return launch_check<double, 3, 2>(a);
    default: return hipErrorNotSupported;
  }
}

hipError_t launch_f64_project(const LaunchArgs& a, const double* a64, int D, int R, int W) {
  F64Args f;
  f.cfgs = a.cfgs; f.tab = static_cast<const double*>(a.tab); f.a64 = a64; f.probs = a.probs; f.items = a.items;
  f.n_items = a.n_items;
  f.xi_bar = static_cast<const double*>(a.xi_bar); f.bvals = static_cast<const double*>(a.bvals);
  f.xi0 = static_cast<const double*>(a.xi0); f.lam0 = static_cast<const double*>(a.lam0); f.iters = a.iters;
  f.xi_out = static_cast<double*>(a.xi_out); f.lam_out = static_cast<double*>(a.lam_out);
  f.resid_out = static_cast<double*>(a.resid_out); f.status_out = a.status_out;
  f.ckpt = static_cast<double*>(a.ckpt); f.ckpt_every = a.ckpt_every; f.ckpt_stride = a.ckpt_stride;
  f.fpr = (a.flags & SF_FP_RESIDUAL) != 0;
  switch (D * 100 + R * 10 + W) {
    case 218: return launch_instance<2, 1, 8>(f, a.lds_bytes, a.stream);
    case 214: return launch_instance<2, 1, 4>(f, a.lds_bytes, a.stream);
    case 224: return launch_instance<2, 2, 4>(f, a.lds_bytes, a.stream);
    case 223: return launch_instance<2, 2, 3>(f, a.lds_bytes, a.stream);
    case 318: return launch_instance<3, 1, 8>(f, a.lds_bytes, a.stream);
    case 314: return launch_instance<3, 1, 4>(f, a.lds_bytes, a.stream);
    case 324: return launch_instance<3, 2, 4>(f, a.lds_bytes, a.stream);
    case 323: return launch_instance<3, 2, 3>(f, a.lds_bytes, a.stream);
    default: return hipErrorNotSupported;
  }
}

}  // namespace sf
