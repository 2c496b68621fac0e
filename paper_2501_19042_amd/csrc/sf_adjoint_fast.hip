// Reverse sweep of the unrolled SF iterations on the matrix cores (fp32), one or more checkpoint segments
// per launch; the segments' forward states are recomputed beforehand by the forward MFMA kernel.
//
// One iteration, in the direct form of eq. (xi_step) (see sf_adjoint.hip for the derivation):
//   Y = F xi,  R = Y - Pi(Y) per constraint block,  g = F^T (rho R),  lambda' = lambda - g,
//   xi' = xi_p + Z S_f Z^T (xi_bar + lambda' - g + G_rho (xi - xi_p)).
// Given the cotangents (gxi', glam') and u = Z S_f Z^T gxi':
//   gxi_bar += u,  glam = glam' + u,  gg = -glam - u,
//   gxi = (gxi' - u on the free coefficients; G_rho u on the pinned ones at k = 0, else 0)
//         + F^T J_R^T (rho F gg),
// with J_R the 3x3 Jacobian of each active block's residual (collision pairs with ||s|| < 1, bound balls
// with ||v|| > vmax, workspace rows with ||s|| > 1); inactive blocks contribute nothing.
//
// One workgroup of W waves per sample.  A lane owns coefficients (axis, k, robot), robot fastest, so that a
// mean over the robots is a sum over an aligned group of 16R lanes; the cotangents stay in its registers and
// the states of the next step are loaded ahead.  An iteration has three barriers: after the cotangents and
// their robot means, after the multiplier cotangent gg, after the tiles' partial back-projections.
// The F and F^T products run as in the forward kernel, per 16-step time tile, and so do the tests that skip
// work whose result is exactly zero: pair lists kept until a robot may have moved by the margin, ball and
// workspace rows skipped while a drift bound proves them inactive (states move little from one step to the
// next in either direction).  The products of gg are formed only for tiles with a listed pair or an active
// row.
//
// What bounds it: the chain of one reverse iteration, at two workgroups per CU.  16 robots x 512 samples: 6.2
// us per iteration, against 12.6 us for a sweep that re-evaluated every box and ball, held the cotangents in
// LDS and took six barriers.  24 robots with a workspace x 48 samples: 9.4 us, against 370 us (recomputation
// included) in the generic adjoint.
#include "sf_fast_kernel.h"
#include "sf_adjoint.h"

namespace sf {
namespace {

using namespace fastk;

// LDS plan (words).  Operands of the products are stored [axis][4 KS coefficients][16R robots], zero past the
// polynomial and the swarm, so that they load without masks.
struct AdjLds {
  int xk, gg, gf, ubar, x1, dx, mx, pairs, tiles, per_wave, total;
  int xt, wt, ct, bb, list;   // inside one wave's region
};

constexpr size_t kAdjLds = 160 * 1024;

__host__ __device__ inline AdjLds adj_fast_plan(const DevCfg& c, int R, int KS, int W) {
  const int NR = 16 * R, Np = c.n * (c.n - 1) / 2, TQ = ((c.H + 15) / 16 + W - 1) / W;
  AdjLds p;
  int o = 0;
  p.xk = o; o += 3 * 4 * KS * NR;           // xi^k
  p.gg = o; o += 3 * 4 * KS * NR;           // multiplier cotangent
  p.gf = o; o += 3 * c.mf * NR;             // cotangents of the free coefficients
  p.ubar = o; o += (3 * c.mf + 3) & ~3;     // their robot means
  p.x1 = o; o += 2 * c.mf * c.mf;           // X1, X01
  p.dx = o; o += 2 * 3 * NR;                // [iteration & 1][axis][robot]: largest change of a coefficient
  p.mx = o; o += 2 * 3 * NR;                // [iteration & 1][row kind][robot]: largest squares of the rows
  p.pairs = o; o += (Np + 1) / 2;           // i | j << 8, 16-bit
  o = (o + 3) & ~3;
  p.xt = 0;                                 // positions of xi^k; later the partial back-projection
  p.wt = 3 * NR * 16;                       // positions of gg
  p.ct = 6 * NR * 16;                       // Jacobian-transpose accumulator, zero between tiles
  p.bb = 9 * NR * 16;                       // boxes
  p.list = p.bb + box_row(R) * NR;          // per tile of the wave: count, pair codes (16-bit)
  p.per_wave = (p.list + (TQ * (Np + 1) + 1) / 2 + 3) & ~3;
  p.tiles = o;
  o += W * p.per_wave;
  p.total = o;
  return p;
}

// Word of coefficient (robot, axis, kk) in a wave's partial back-projection, stored as the products leave it:
// [axis][robot tile][r][lane], lane (col, grp) = (robot, coefficient grp + 4 r).
template <int R>
__device__ __forceinline__ int part_at(int robot, int d, int kk) {
  return ((d * R + (robot >> 4)) * 4 + (kk >> 2)) * 64 + (kk & 3) * 16 + (robot & 15);
}

// Y[rr][d] = basis rows x coefficients for one tile: lane (col, grp) gets robot 16 rr + col at times 4 grp + r.
template <int R, int KS>
__device__ __forceinline__ void tile_product(const float4 av, const float* src, int lane, f4 (&Y)[R][3]) {
  constexpr int NR = 16 * R;
  const float a1[4] = {av.x, av.y, av.z, av.w};
  const float* sp = src + (lane >> 4) * NR + (lane & 15);
#pragma unroll
  for (int rr = 0; rr < R; ++rr)
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = 0; s < KS; ++s) acc = mfma4(a1[s], sp[(d * 4 * KS + 4 * s) * NR + 16 * rr], acc);
      Y[rr][d] = acc;
    }
}

template <int R>
__device__ __forceinline__ void store_tile(float* buf, int lane, const f4 (&Y)[R][3]) {
#pragma unroll
  for (int rr = 0; rr < R; ++rr)
#pragma unroll
    for (int d = 0; d < 3; ++d)
      *reinterpret_cast<f4*>(buf + tile_at(d * 16 * R + 16 * rr + (lane & 15), 4 * (lane >> 4))) = Y[rr][d];
}

// Boxes of a tile's positions into bb.
template <int R>
__device__ __forceinline__ void store_boxes(float* bb, int lane, const f4 (&Y)[R][3]) {
#pragma unroll
  for (int rr = 0; rr < R; ++rr) {
    float lo[3], hi[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const f4 v = Y[rr][d];
      lo[d] = grp_min(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])));
      hi[d] = grp_max(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
    }
    if ((lane >> 4) == 0) {
      float* bq = bb + (16 * rr + (lane & 15)) * box_row(R);
      *reinterpret_cast<f4*>(bq) = f4{lo[0], lo[1], lo[2], 0.0f};
      *reinterpret_cast<f4*>(bq + 4) = f4{hi[0], hi[1], hi[2], 0.0f};
    }
  }
}

// Lists the pairs whose boxes, each gap shrunk by the margins, are closer than the safety distance (1e-4
// relative slack); returns their number (uniform).
template <int R>
__device__ __forceinline__ int list_pairs(const float* bb, const uint16_t* pairs, int Np, int lane, float mgx, float mgz,
                                          float ia2, float ib2, uint16_t* list) {
  int count = 0;
  for (int base = 0; base < Np; base += 64) {
    const int p = base + lane;
    const int code = pairs[min(p, Np - 1)], i = code & 255, j = code >> 8;
    const f4 li = *reinterpret_cast<const f4*>(bb + i * box_row(R));
    const f4 hi = *reinterpret_cast<const f4*>(bb + i * box_row(R) + 4);
    const f4 lj = *reinterpret_cast<const f4*>(bb + j * box_row(R));
    const f4 hj = *reinterpret_cast<const f4*>(bb + j * box_row(R) + 4);
    float g2 = 0.0f;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const float gap = fmaxf(0.0f, fmaxf(lj[d] - hi[d], li[d] - hj[d]) - (d == 2 ? mgz : mgx));
      g2 += gap * gap * (d == 2 ? ib2 : ia2);
    }
    const bool act = p < Np && g2 < 1.0001f;
    const uint64_t mask = ballot(act);
    if (act) list[count + lanes_below(mask)] = (uint16_t)code;
    count += __popcll(mask);
  }
  return count;
}

// Items of a lane: coefficients (axis d, kk, robot), robot fastest, t = tid + j * 64 W.
struct Item {
  int q, row, part, d, kk, rb;   // index in the sample (-1: none), word in the operands, word in the partials
};
template <int R, int KS>
__device__ __forceinline__ Item make_item(int t, int n, int m) {
  constexpr int NR = 16 * R;
  Item i;
  i.rb = t % NR;
  i.kk = (t / NR) % m;
  i.d = t / (NR * m);
  const bool ok = i.d < 3 && i.rb < n;
  i.q = ok ? (i.rb * 3 + i.d) * m + i.kk : -1;
  i.row = ok ? (i.d * 4 * KS + i.kk) * NR + i.rb : 0;
  i.part = ok ? part_at<R>(i.rb, i.d, i.kk) : 0;
  if (i.d >= 3) i.d = 2;
  return i;
}

// (two waves per SIMD: two workgroups of four waves, or one of six or eight, per CU)
template <int R, int KS, int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2, 2))) adjoint_fast_kernel(AdjFastArgs A) {
  extern __shared__ __align__(16) float smem[];
  constexpr int NR = 16 * R, nthr = 64 * W;
  constexpr int NI = (3 * 4 * KS * NR + nthr - 1) / nthr;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float4* a32 = static_cast<const float4*>(A.a32);
  const int64_t stride = A.stride;
  for (int it = blockIdx.x; it < A.n_items; it += gridDim.x) {
    const WorkItem w = A.items[it];
    const DevProblem pr = A.probs[w.problem];
    const DevCfg& c = A.cfgs[pr.cfg];
    const AdjLds Lp = adj_fast_plan(c, R, KS, W);
    const int n = c.n, m = c.m, mf = c.mf, H = c.H, nDm = n * 3 * m;
    const int Np = n * (n - 1) / 2, NT = (H + 15) / 16, TQ = (NT + W - 1) / W;
    const float* Gfx = A.tab + c.off_Gfx;
    const float* Rfx = A.tab + c.off_Rfx;
    const float ia2 = (float)c.inv_a2, ib2 = (float)c.inv_b2;
    const float vmax = (float)c.vmax, amax = (float)c.amax, Lv = (float)c.lip_v, La = (float)c.lip_a;
    const float n_rho_c = (float)c.n_rho_c, inv_n = 1.0f / (float)n;
    const bool ws_on = c.ws_on != 0;
    const float wcx = c.ws_f[0], wcy = c.ws_f[1], wcz = c.ws_f[2], wia2 = c.ws_f[3], wib2 = c.ws_f[4], wsc = c.ws_f[5];
    const int on = (c.vel_on ? 1 : 0) | (c.acc_on ? 2 : 0) | (ws_on ? 4 : 0);
    const float skx = (float)(c.skin * c.a) * 0.999f, skz = (float)(c.skin * c.b) * 0.999f;
    const float4* a32c = a32 + c.off_a32;
    float *sxk = smem + Lp.xk, *sgg = smem + Lp.gg, *sgf = smem + Lp.gf, *subar = smem + Lp.ubar;
    float *sX1 = smem + Lp.x1, *sX01 = sX1 + mf * mf;
    // fp32 bits: non-negative floats order like their bits, and a NaN lies above all of them
    uint32_t* sdx = reinterpret_cast<uint32_t*>(smem + Lp.dx);
    uint32_t* smx = reinterpret_cast<uint32_t*>(smem + Lp.mx);
    uint16_t* spairs = reinterpret_cast<uint16_t*>(smem + Lp.pairs);
    float* wbuf = smem + Lp.tiles + wave * Lp.per_wave;
    float *Xt = wbuf + Lp.xt, *Wt = wbuf + Lp.wt, *Ct = wbuf + Lp.ct, *bb = wbuf + Lp.bb;
    uint16_t* lists = reinterpret_cast<uint16_t*>(wbuf + Lp.list);
    {
      const int tid = threadIdx.x;
      for (int q = tid; q < n * n; q += nthr) {
        const int i = q / n, j = q - i * n;
        if (j > i) spairs[i * n - i * (i + 1) / 2 + j - i - 1] = (uint16_t)(i | (j << 8));
      }
      for (int q = tid; q < mf * mf; q += nthr) {
        sX1[q] = (A.tab + c.off_X1)[q];
        sX01[q] = (A.tab + c.off_X01)[q];
      }
      for (int q = tid; q < 3 * 4 * KS * NR; q += nthr) sxk[q] = sgg[q] = 0.0f;
      for (int q = tid & 63; q < 3 * NR * 16; q += 64) Ct[q] = 0.0f;
    }
    Item im[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) im[j] = make_item<R, KS>(threadIdx.x + j * nthr, n, m);

    for (int sl = w.first; sl < w.first + w.count; ++sl) {
      const int64_t coef = pr.coef_off + (int64_t)sl * nDm;
      const float wf = A.w_fpr ? A.w_fpr[pr.sample_base + sl] : 0.0f;
      float* cg = A.carry + coef;
      // cotangents of the lane's coefficients, and the states of the next step
      float gxi[NI], glam[NI], gxb[NI], x0[NI], x1[NI], l0[NI], l1[NI];
      auto fetch = [&](int k) {
        const int seg = k / A.every;
        const float* s = A.states + ((int64_t)(seg - A.seg0) * (A.every + 1) + (k - seg * A.every)) * 2 * stride + coef;
#pragma unroll
        for (int j = 0; j < NI; ++j)
          if (im[j].q >= 0) {
            x0[j] = s[im[j].q];
            x1[j] = s[2 * stride + im[j].q];
            if (wf != 0.0f) {
              l0[j] = s[stride + im[j].q];
              l1[j] = s[3 * stride + im[j].q];
            }
          }
      };
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int q = im[j].q;
        x0[j] = x1[j] = l0[j] = l1[j] = 0.0f;
        gxi[j] = q < 0 ? 0.0f : (A.init ? (A.g_xi_out ? A.g_xi_out[coef + q] : 0.0f) : cg[q]);
        glam[j] = q < 0 ? 0.0f : (A.init ? (A.g_lam_out ? A.g_lam_out[coef + q] : 0.0f) : cg[stride + q]);
        gxb[j] = q < 0 || A.init ? 0.0f : cg[2 * stride + q];
      }
      for (int q = threadIdx.x; q < 2 * 3 * NR; q += nthr) sdx[q] = smx[q] = 0u;
      fetch(A.k_end - 1);
      // per robot (lane), identical in every wave: slack to the bounds at the last evaluation less the drift
      // since, and drift since the pair lists were built
      float sv = -1.0f, sacc = -1.0f, sws = -1.0f, px = 0.0f, py = 0.0f, pz = 0.0f;
      int prev_eval = 0;
      __syncthreads();
      for (int k = A.k_end - 1; k >= A.k_begin; --k) {
        // (per-lane indices from an opaque copy: keeps per-lane addresses next to their uses)
        int tid_k = threadIdx.x;
        asm volatile("" : "+v"(tid_k));
        const int tid = tid_k, lane = tid_k & 63, col = lane & 15, grp = lane >> 4;
        const int par = k & 1;
        // the first step of a launch and of a segment (whose states are recomputed on their own) starts afresh
        const bool fresh = k == A.k_end - 1 || (k + 1) % A.every == 0;
        float dfx[NI], dfl[NI];
        // z^{k+1}'s share of the fixed-point residual term; xi^k, the free cotangents and their robot means
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          if (tid - lane + j * nthr >= 3 * m * NR) break;   // (uniform over the wave)
          const Item& t = im[j];
          dfx[j] = x1[j] - x0[j];
          dfl[j] = l1[j] - l0[j];
          if (wf != 0.0f) {
            gxi[j] += 2.0f * wf * dfx[j];
            glam[j] += 2.0f * wf * dfl[j];
          }
          const int f = t.kk - 3;
          const bool fre = f >= 0 && f < mf;
          if (t.q >= 0) {
            sxk[t.row] = x0[j];
            atomicMax(sdx + (par * 3 + t.d) * NR + t.rb, __float_as_uint(fabsf(dfx[j])));
            if (fre) sgf[(t.d * mf + f) * NR + t.rb] = gxi[j];
          }
          const float mean = group_sum<NR>(t.q >= 0 ? gxi[j] : 0.0f) * inv_n;
          if (fre && t.rb == 0 && t.q >= 0) subar[t.d * mf + f] = mean;
        }
        __syncthreads();
        // u = Z S_f Z^T gxi, and the multiplier cotangent gg
        float uu[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          uu[j] = 0.0f;
          const Item& t = im[j];
          const int f = t.kk - 3;
          if (t.q >= 0) {
            if (f >= 0 && f < mf) {
              float u = 0.0f;
#pragma unroll 5
              for (int f2 = 0; f2 < mf; ++f2) {
                u = fmaf(sX1[f * mf + f2], sgf[(t.d * mf + f2) * NR + t.rb], u);
                u = fmaf(sX01[f * mf + f2], subar[t.d * mf + f2], u);
              }
              uu[j] = u;
              gxi[j] -= u;
            } else {
              gxi[j] = 0.0f;   // (its cotangent at k = 0 is added below)
            }
            gxb[j] += uu[j];
            const float gl = glam[j] + uu[j];
            glam[j] = gl;
            sgg[t.row] = -gl - uu[j];
          }
        }
        for (int q = tid; q < 3 * NR; q += nthr) {
          sdx[(par ^ 1) * 3 * NR + q] = 0u;
          smx[par * 3 * NR + q] = 0u;
        }
        __syncthreads();
        if (k > A.k_begin) fetch(k - 1);
        if (k == 0) {   // pinned coefficients: G_rho u restricted to them
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            if (tid - lane + j * nthr >= 3 * m * NR) break;
            const Item& t = im[j];
            const int f = t.kk - 3;
            const bool fre = f >= 0 && f < mf;
            if (t.q >= 0 && fre) sgf[(t.d * mf + f) * NR + t.rb] = uu[j];
            const float mean = group_sum<NR>(t.q >= 0 ? uu[j] : 0.0f) * inv_n;
            if (fre && t.rb == 0 && t.q >= 0) subar[t.d * mf + f] = mean;
          }
          __syncthreads();
#pragma unroll
          for (int j = 0; j < NI; ++j) {
            const Item& t = im[j];
            const int f = t.kk - 3, r6 = t.kk < 3 ? t.kk : t.kk - (m - kNFix);
            if (t.q >= 0 && !(f >= 0 && f < mf)) {
              float v = 0.0f;
              for (int f2 = 0; f2 < mf; ++f2) {
                const float u2 = sgf[(t.d * mf + f2) * NR + t.rb];
                v = fmaf(n_rho_c * Gfx[f2 * kNFix + r6], u2 - subar[t.d * mf + f2], v);
                v = fmaf(Rfx[f2 * kNFix + r6], u2, v);
              }
              gxi[j] = v;
            }
          }
        }
        // what to evaluate (see the forward kernel): a row moves between two states by at most its basis'
        // largest row sum times the largest change of a coefficient
        int eval = 7;
        bool rebuild = true;
        {
          bool ev = false, ea = false, ew = false, er = false;
          if (lane < n) {
            const uint32_t* pm = smx + (par ^ 1) * 3 * NR + lane;
            if (prev_eval & 1) sv = vmax - __builtin_amdgcn_sqrtf(__uint_as_float(pm[0]));
            if (prev_eval & 2) sacc = amax - __builtin_amdgcn_sqrtf(__uint_as_float(pm[NR]));
            if (prev_eval & 4) sws = 1.0f - __builtin_amdgcn_sqrtf(__uint_as_float(pm[2 * NR]));
            const float d0 = __uint_as_float(sdx[(par * 3 + 0) * NR + lane]);
            const float d1 = __uint_as_float(sdx[(par * 3 + 1) * NR + lane]);
            const float d2 = __uint_as_float(sdx[(par * 3 + 2) * NR + lane]);
            const float dn = __builtin_amdgcn_sqrtf(d0 * d0 + d1 * d1 + d2 * d2);
            px = drift_add(px, d0);
            py = drift_add(py, d1);
            pz = drift_add(pz, d2);
            sv = slack_less(sv, Lv * dn);
            sacc = slack_less(sacc, La * dn);
            if (ws_on) sws = slack_less(sws, __builtin_amdgcn_sqrtf((d0 * d0 + d1 * d1) * wia2 + d2 * d2 * wib2));
            er = !(px <= skx && py <= skx && pz <= skz);
            ev = !(sv > 1e-4f * vmax);
            ea = !(sacc > 1e-4f * amax);
            ew = !(sws > 1e-4f);
          }
          if (!fresh) {
            eval = (ballot(ev) ? 1 : 0) | (ballot(ea) ? 2 : 0) | (ballot(ew) ? 4 : 0);
            rebuild = ballot(er) != 0;
          }
          eval &= on;
          prev_eval = eval;
        }
        float mgx = 0.0f, mgz = 0.0f;
        if (rebuild) {
          // twice the drift margin plus the rounding of a position: 2^-16 of a bound on the coefficients until
          // the next rebuild
          px = py = pz = 0.0f;
          float cm = 0.0f;
          for (int q = lane; q < 3 * 4 * KS * NR; q += 64) cm = fmaxf(cm, fabsf(sxk[q]));
          const float tol = 1.52587890625e-5f * (wave_max(cm) + fmaxf(skx, skz));
          mgx = 2.0f * skx + tol;
          mgz = 2.0f * skz + tol;
        }
        // ---- F^T J_R^T (rho F gg) over this wave's time tiles ----
        f4 gacc[R][3];
        float vm[3][R];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
#pragma unroll
          for (int d = 0; d < 3; ++d) gacc[rr][d] = f4{0.0f, 0.0f, 0.0f, 0.0f};
          vm[0][rr] = vm[1][rr] = vm[2][rr] = 0.0f;
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
            f4 Y[R][3];
            const float4 av = a32c[((tau * 3) * 2) * 64 + lane];
            tile_product<R, KS>(av, sxk, lane, Y);
            store_tile<R>(Xt, lane, Y);
            if (rebuild) {
              store_boxes<R>(bb, lane, Y);
              wave_sync();
              count = list_pairs<R>(bb, spairs, Np, lane, mgx, mgz, ia2, ib2, tl + 1);
              if (lane == 0) tl[0] = (uint16_t)count;
            }
            count = __builtin_amdgcn_readfirstlane(count);
            if (eval & 4) {
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const float qx = Y[rr][0][r] - wcx, qy = Y[rr][1][r] - wcy, qz = Y[rr][2][r] - wcz;
                  const float s2 = (qx * qx + qy * qy) * wia2 + qz * qz * wib2;
                  vm[2][rr] = s2 > vm[2][rr] || s2 != s2 ? s2 : vm[2][rr];
                  wnz |= 16 * rr + col < n && s2 > 1.0f;
                }
              wnz = ballot(wnz) != 0;
            }
            if (count > 0 || wnz) {
              f4 G[R][3];
              tile_product<R, KS>(av, sgg, lane, G);
              if (count > 0) store_tile<R>(Wt, lane, G);
              if (wnz) {
                // J^T w of the workspace rows, scaled by rho_w / rho_c so that it joins the pairs' accumulator
                // (zero until now)
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int r = 0; r < 4; ++r) {
                    const float qx = Y[rr][0][r] - wcx, qy = Y[rr][1][r] - wcy, qz = Y[rr][2][r] - wcz;
                    const float s2 = (qx * qx + qy * qy) * wia2 + qz * qz * wib2;
                    float jx = 0.0f, jy = 0.0f, jz = 0.0f;
                    if (16 * rr + col < n && s2 > 1.0f) {
                      const float rs = rsqrtf(s2), f = wsc * (1.0f - rs);
                      const float k3 = wsc * rs * rs * rs * (qx * G[rr][0][r] + qy * G[rr][1][r] + qz * G[rr][2][r]);
                      jx = f * G[rr][0][r] + k3 * qx * wia2;
                      jy = f * G[rr][1][r] + k3 * qy * wia2;
                      jz = f * G[rr][2][r] + k3 * qz * wib2;
                    }
                    Y[rr][0][r] = jx;
                    Y[rr][1][r] = jy;
                    Y[rr][2][r] = jz;
                  }
                store_tile<R>(Ct, lane, Y);
              }
            }
            wave_sync();
          }
          // Jacobian-transpose products of the active pair-times (lanes cover (pair, time) items)
          const int tsh = nt <= 4 ? 2 : (nt <= 8 ? 3 : 4);
          const int tt = lane & ((1 << tsh) - 1), ps = lane >> tsh, ppr = 64 >> tsh;
          bool nzc = false;
          for (int base = 0; base < count; base += ppr) {
            const int slot = base + ps;
            if (slot < count && tt < nt) {
              const int pij = tl[1 + slot], i = pij & 255, j = pij >> 8;
              const float rx = Xt[tile_at(i, tt)] - Xt[tile_at(j, tt)];
              const float ry = Xt[tile_at(NR + i, tt)] - Xt[tile_at(NR + j, tt)];
              const float rz = Xt[tile_at(2 * NR + i, tt)] - Xt[tile_at(2 * NR + j, tt)];
              const float ss = (rx * rx + ry * ry) * ia2 + rz * rz * ib2;
              if (ss >= FLT_MIN && ss < 1.0f) {
                const float vx = Wt[tile_at(i, tt)] - Wt[tile_at(j, tt)];
                const float vy = Wt[tile_at(NR + i, tt)] - Wt[tile_at(NR + j, tt)];
                const float vz = Wt[tile_at(2 * NR + i, tt)] - Wt[tile_at(2 * NR + j, tt)];
                const float rs = rsqrtf(ss), f = 1.0f - rs;
                const float k3 = rs * rs * rs * (rx * vx + ry * vy + rz * vz);
                const float jx = f * vx + k3 * rx * ia2, jy = f * vy + k3 * ry * ia2, jz = f * vz + k3 * rz * ib2;
                nzc = true;
                atomicAdd(Ct + tile_at(i, tt), jx);
                atomicAdd(Ct + tile_at(NR + i, tt), jy);
                atomicAdd(Ct + tile_at(2 * NR + i, tt), jz);
                atomicAdd(Ct + tile_at(j, tt), -jx);
                atomicAdd(Ct + tile_at(NR + j, tt), -jy);
                atomicAdd(Ct + tile_at(2 * NR + j, tt), -jz);
              }
            }
          }
          if (wnz || ballot(nzc) != 0) {
            wave_sync();
            const float4 bq = a32c[((tau * 3) * 2 + 1) * 64 + lane];   // rho_c P (zero past the horizon)
            const float b4[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                f4* cp = reinterpret_cast<f4*>(Ct + tile_at(d * NR + 16 * rr + col, 4 * grp));
                const f4 cr = *cp;
                *cp = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int s = 0; s < 4; ++s) gacc[rr][d] = mfma4(b4[s], cr[s], gacc[rr][d]);
              }
          }
          wave_sync();
          // bound balls: J^T (F_b gg) where ||F_b xi^k|| exceeds the bound
#pragma unroll
          for (int b = 1; b < 3; ++b) {
            if (!(eval & b)) continue;
            const float lim = b == 1 ? vmax : amax;
            const float4 av = a32c[((tau * 3 + b) * 2) * 64 + lane];
            f4 V[R][3];
            tile_product<R, KS>(av, sxk, lane, V);
            bool nz = false;
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float ss = V[rr][0][r] * V[rr][0][r] + V[rr][1][r] * V[rr][1][r] + V[rr][2][r] * V[rr][2][r];
                vm[b - 1][rr] = ss > vm[b - 1][rr] || ss != ss ? ss : vm[b - 1][rr];
                nz |= ss > lim * lim;
              }
            if (ballot(nz) == 0) continue;
            f4 G[R][3];
            tile_product<R, KS>(av, sgg, lane, G);
            const float4 bq = a32c[((tau * 3 + b) * 2 + 1) * 64 + lane];   // rho_b P_b
            const float b4[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float vx = V[rr][0][r], vy = V[rr][1][r], vz = V[rr][2][r];
                const float gx = G[rr][0][r], gy = G[rr][1][r], gz = G[rr][2][r];
                const float ss = vx * vx + vy * vy + vz * vz;
                float jx = 0.0f, jy = 0.0f, jz = 0.0f;
                if (ss > lim * lim) {
                  const float rs = rsqrtf(ss), h = 1.0f - lim * rs;
                  const float k3 = lim * rs * rs * rs * (vx * gx + vy * gy + vz * gz);
                  jx = h * gx + k3 * vx;
                  jy = h * gy + k3 * vy;
                  jz = h * gz + k3 * vz;
                }
                V[rr][0][r] = jx;
                V[rr][1][r] = jy;
                V[rr][2][r] = jz;
              }
#pragma unroll
              for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int s = 0; s < 4; ++s) gacc[rr][d] = mfma4(b4[s], V[rr][d][s], gacc[rr][d]);
            }
          }
        }
        // this wave's partial back-projection and row maxima
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int r = 0; r < 4; ++r) Xt[((d * R + rr) * 4 + r) * 64 + lane] = gacc[rr][d][r];
#pragma unroll
        for (int b = 0; b < 3; ++b)
          if (eval & (1 << b)) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr) atomicMax(smx + (par * 3 + b) * NR + 16 * rr + col, __float_as_uint(vm[b][rr]));
          }
        __syncthreads();
        const float* parts = smem + Lp.tiles;
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const Item& t = im[j];
          if (t.q < 0) continue;
          float g = gxi[j];
#pragma unroll
          for (int ww = 0; ww < W; ++ww) g += parts[ww * Lp.per_wave + t.part];
          if (A.pend && k == A.iters - 1) g += A.pend[coef + t.q];
          if (wf != 0.0f) {   // z^k's share of the fixed-point residual term
            g -= 2.0f * wf * dfx[j];
            glam[j] -= 2.0f * wf * dfl[j];
          }
          gxi[j] = g;
        }
      }
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int q = im[j].q;
        if (q < 0) continue;
        if (A.last) {
          if (A.g_xi0) A.g_xi0[coef + q] = gxi[j];
          if (A.g_lam0) A.g_lam0[coef + q] = glam[j];
          if (A.g_xi_bar) A.g_xi_bar[coef + q] = gxb[j];
        } else {
          cg[q] = gxi[j];
          cg[stride + q] = glam[j];
          cg[2 * stride + q] = gxb[j];
        }
      }
      __syncthreads();
    }
  }
}

// Final-residual term, g_resid ||r_p^K||^2 with r_p = F xi^K - e(F xi^{K-1}) = D + R (D = F (xi^K - xi^{K-1}),
// R the blocks' residuals at xi^{K-1}): with q = 2 g_resid (D + R) per block, its cotangent of xi^K is F^T q
// and that of xi^{K-1} F^T (J_R^T q - q).  Over the pairs of robot i the part without R sums to
// n D_i - sum_j D_j, so only listed pairs are visited: once for R, once for J_R^T q.  One workgroup of four
// waves per sample writes the carries (gxi, glam, gxb) and pend; the previous kernel, which formed every pair
// from the basis rows in global memory, took 224 us at 16 robots x 512 samples, this one 25 us.
template <int R, int KS>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) adjoint_resid_kernel(AdjFastArgs A) {
  extern __shared__ __align__(16) float smem[];
  constexpr int NR = 16 * R, W = 4, nthr = 64 * W;
  constexpr int NI = (3 * 4 * KS * NR + nthr - 1) / nthr;
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t stride = A.stride;
  for (int it = blockIdx.x; it < A.n_items; it += gridDim.x) {
    const WorkItem w = A.items[it];
    const DevProblem pr = A.probs[w.problem];
    const DevCfg& c = A.cfgs[pr.cfg];
    const AdjLds Lp = adj_fast_plan(c, R, KS, W);
    const int n = c.n, m = c.m, H = c.H, nDm = n * 3 * m, Np = n * (n - 1) / 2, NT = (H + 15) / 16;
    const float ia2 = (float)c.inv_a2, ib2 = (float)c.inv_b2, sb = (float)c.b;
    const bool ws_on = c.ws_on != 0;
    const float wcx = c.ws_f[0], wcy = c.ws_f[1], wcz = c.ws_f[2], wia2 = c.ws_f[3], wib2 = c.ws_f[4];
    // (the S4 operands carry rho; these rows are unweighted)
    const float wgt[3] = {(float)(1.0 / c.rho_c), c.vel_on ? (float)(1.0 / c.rho_v) : 0.0f,
                          c.acc_on ? (float)(1.0 / c.rho_a) : 0.0f};
    const float4* a32c = static_cast<const float4*>(A.a32) + c.off_a32;
    float *sxk = smem + Lp.xk, *sdl = smem + Lp.gg;   // xi^{K-1}, xi^K - xi^{K-1}
    uint16_t* spairs = reinterpret_cast<uint16_t*>(smem + Lp.pairs);
    float* wbuf = smem + Lp.tiles + wave * Lp.per_wave;
    float *Xt = wbuf + Lp.xt, *Wt = wbuf + Lp.wt, *Ct = wbuf + Lp.ct, *bb = wbuf + Lp.bb;
    uint16_t* tl = reinterpret_cast<uint16_t*>(wbuf + Lp.list);
    for (int q = tid; q < n * n; q += nthr) {
      const int i = q / n, j = q - i * n;
      if (j > i) spairs[i * n - i * (i + 1) / 2 + j - i - 1] = (uint16_t)(i | (j << 8));
    }
    for (int q = tid; q < 3 * 4 * KS * NR; q += nthr) sxk[q] = sdl[q] = 0.0f;
    __syncthreads();
    for (int sl = w.first; sl < w.first + w.count; ++sl) {
      const int64_t coef = pr.coef_off + (int64_t)sl * nDm;
      const float gres = A.g_resid[pr.sample_base + sl];
      const float g2r = 2.0f * gres;
      // states of the last iteration
      const int seg = (A.iters - 1) / A.every;
      const float* xs = A.states + ((int64_t)(seg - A.seg0) * (A.every + 1) + (A.iters - 1 - seg * A.every)) * 2 * stride + coef;
      Item im[NI];
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        im[j] = make_item<R, KS>(tid + j * nthr, n, m);
        if (im[j].q >= 0) {
          const float x0 = xs[im[j].q];
          sxk[im[j].row] = x0;
          sdl[im[j].row] = xs[2 * stride + im[j].q] - x0;
        }
      }
      for (int q = lane; q < 3 * NR * 16; q += 64) Ct[q] = 0.0f;
      __syncthreads();
      f4 ga[R][3], gj[R][3];   // F^T q, F^T J_R^T q
#pragma unroll
      for (int rr = 0; rr < R; ++rr)
#pragma unroll
        for (int d = 0; d < 3; ++d) ga[rr][d] = gj[rr][d] = f4{0.0f, 0.0f, 0.0f, 0.0f};
      float cm = 0.0f;
      for (int q = lane; q < 3 * 4 * KS * NR; q += 64) cm = fmaxf(cm, fabsf(sxk[q]));
      const float tol = 1.52587890625e-5f * wave_max(cm);
#pragma unroll 1
      for (int tau = wave; tau < (gres != 0.0f ? NT : 0); tau += W) {
        const int nt = min(16, H - 16 * tau);
#pragma unroll 1
        for (int b = 0; b < 3; ++b) {
          if (b > 0 && !(b == 1 ? c.vel_on : c.acc_on)) continue;
          const float4 av = a32c[((tau * 3 + b) * 2) * 64 + lane];
          const float4 bq = a32c[((tau * 3 + b) * 2 + 1) * 64 + lane];
          const float wb = b == 0 ? wgt[0] : (b == 1 ? wgt[1] : wgt[2]);
          const float b4[4] = {bq.x * wb, bq.y * wb, bq.z * wb, bq.w * wb};
          auto back = [&](const f4 (&v)[R][3], f4 (&g)[R][3]) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int s = 0; s < 4; ++s) g[rr][d] = mfma4(b4[s], v[rr][d][s], g[rr][d]);
          };
          f4 Y[R][3], D[R][3];
          tile_product<R, KS>(av, sxk, lane, Y);
          tile_product<R, KS>(av, sdl, lane, D);
          if (b > 0) {
            const float lim = b == 1 ? (float)c.vmax : (float)c.amax;
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float vx = Y[rr][0][r], vy = Y[rr][1][r], vz = Y[rr][2][r];
                const float ss = vx * vx + vy * vy + vz * vz;
                const bool act = ss > lim * lim;
                const float rs = act ? rsqrtf(ss) : 0.0f, h = act ? 1.0f - lim * rs : 0.0f;
                const float qx = g2r * (D[rr][0][r] + h * vx), qy = g2r * (D[rr][1][r] + h * vy),
                            qz = g2r * (D[rr][2][r] + h * vz);
                const float k3 = act ? lim * rs * rs * rs * (vx * qx + vy * qy + vz * qz) : 0.0f;
                D[rr][0][r] = qx;
                D[rr][1][r] = qy;
                D[rr][2][r] = qz;
                Y[rr][0][r] = act ? h * qx + k3 * vx : 0.0f;
                Y[rr][1][r] = act ? h * qy + k3 * vy : 0.0f;
                Y[rr][2][r] = act ? h * qz + k3 * vz : 0.0f;
              }
            back(D, ga);
            back(Y, gj);
            continue;
          }
          store_tile<R>(Xt, lane, Y);
          store_tile<R>(Wt, lane, D);
          store_boxes<R>(bb, lane, Y);
          wave_sync();
          const int count = list_pairs<R>(bb, spairs, Np, lane, tol, tol, ia2, ib2, tl + 1);
          // the pairs' part without R, and the workspace rows
          f4 S[R][3];
#pragma unroll
          for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              float s = group_sum<16>(D[0][d][r]);
              if constexpr (R == 2) s += group_sum<16>(D[R - 1][d][r]);
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
                S[rr][d][r] = 16 * rr + col < n ? g2r * ((float)n * D[rr][d][r] - s) : 0.0f;
            }
          if (ws_on) {
            f4 J[R][3];
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float px = Y[rr][0][r] - wcx, py = Y[rr][1][r] - wcy, pz = Y[rr][2][r] - wcz;
                const float s2 = (px * px + py * py) * wia2 + pz * pz * wib2;
                const bool real = 16 * rr + col < n, act = real && s2 > 1.0f;
                const float rs = act ? rsqrtf(s2) : 0.0f, f = act ? 1.0f - rs : 0.0f;
                const float qx = real ? g2r * (D[rr][0][r] + f * px) : 0.0f, qy = real ? g2r * (D[rr][1][r] + f * py) : 0.0f,
                            qz = real ? g2r * (D[rr][2][r] + f * pz) : 0.0f;
                const float k3 = rs * rs * rs * (px * qx + py * qy + pz * qz);
                S[rr][0][r] += qx;
                S[rr][1][r] += qy;
                S[rr][2][r] += qz;
                J[rr][0][r] = act ? f * qx + k3 * px * wia2 : 0.0f;
                J[rr][1][r] = act ? f * qy + k3 * py * wia2 : 0.0f;
                J[rr][2][r] = act ? f * qz + k3 * pz * wib2 : 0.0f;
              }
            back(J, gj);
          }
          back(S, ga);
          // listed pairs: 2 g_resid R into F^T q, then J_R^T q
          const int tsh = nt <= 4 ? 2 : (nt <= 8 ? 3 : 4);
          const int tt = lane & ((1 << tsh) - 1), ps = lane >> tsh, ppr = 64 >> tsh;
#pragma unroll 1
          for (int pass = 0; pass < 2 && count > 0; ++pass) {
            wave_sync();
            for (int base = 0; base < count; base += ppr) {
              const int slot = base + ps;
              if (slot < count && tt < nt) {
                const int pij = tl[1 + slot], i = pij & 255, j = pij >> 8;
                float r[3], v[3], Rr[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                  r[d] = Xt[tile_at(d * NR + i, tt)] - Xt[tile_at(d * NR + j, tt)];
                  v[d] = Wt[tile_at(d * NR + i, tt)] - Wt[tile_at(d * NR + j, tt)];
                }
                const float ss = (r[0] * r[0] + r[1] * r[1]) * ia2 + r[2] * r[2] * ib2;
                coll_resid3(r[0], r[1], r[2], ia2, ib2, sb, Rr[0], Rr[1], Rr[2]);
                bool add = Rr[0] != 0.0f || Rr[1] != 0.0f || Rr[2] != 0.0f;
                float o[3];
                if (pass == 0) {
#pragma unroll
                  for (int d = 0; d < 3; ++d) o[d] = g2r * Rr[d];
                } else {
                  add = ss >= FLT_MIN && ss < 1.0f;
                  const float rs = add ? rsqrtf(ss) : 0.0f, f = 1.0f - rs;
                  float rv = 0.0f;
#pragma unroll
                  for (int d = 0; d < 3; ++d) {
                    v[d] = g2r * (v[d] + Rr[d]);
                    rv += r[d] * v[d];
                  }
#pragma unroll
                  for (int d = 0; d < 3; ++d) o[d] = f * v[d] + rs * rs * rs * rv * r[d] * (d == 2 ? ib2 : ia2);
                }
                if (add) {
#pragma unroll
                  for (int d = 0; d < 3; ++d) {
                    atomicAdd(Ct + tile_at(d * NR + i, tt), o[d]);
                    atomicAdd(Ct + tile_at(d * NR + j, tt), -o[d]);
                  }
                }
              }
            }
            wave_sync();
            f4 C[R][3];
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                f4* cp = reinterpret_cast<f4*>(Ct + tile_at(d * NR + 16 * rr + col, 4 * grp));
                C[rr][d] = *cp;
                *cp = f4{0.0f, 0.0f, 0.0f, 0.0f};
              }
            if (pass == 0) back(C, ga);
            else back(C, gj);
          }
          wave_sync();
        }
      }
      // partials of both, then their sums in wave order
#pragma unroll
      for (int d = 0; d < 3; ++d)
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            Xt[((d * R + rr) * 4 + r) * 64 + lane] = ga[rr][d][r];
            Wt[((d * R + rr) * 4 + r) * 64 + lane] = gj[rr][d][r];
          }
      __syncthreads();
      const float* parts = smem + Lp.tiles;
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int q = im[j].q;
        if (q < 0) continue;
        float a = 0.0f, b = 0.0f;
#pragma unroll
        for (int ww = 0; ww < W; ++ww) {
          a += parts[ww * Lp.per_wave + Lp.xt + im[j].part];
          b += parts[ww * Lp.per_wave + Lp.wt + im[j].part];
        }
        A.carry[coef + q] = (A.g_xi_out ? A.g_xi_out[coef + q] : 0.0f) + a;
        A.carry[stride + coef + q] = A.g_lam_out ? A.g_lam_out[coef + q] : 0.0f;
        A.carry[2 * stride + coef + q] = 0.0f;
        A.pend_out[coef + q] = b - a;
      }
      __syncthreads();
    }
  }
}

template <typename K>
hipError_t launch(K kern, const AdjFastArgs& a, int threads, size_t lds) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.n_items), dim3(threads), lds, a.stream, a);
  return hipGetLastError();
}

// Waves per sample: with one robot tile 8 (one time tile per wave up to a horizon of 128) while every sample
// has a CU of its own, else 4, which keeps two samples per CU; with two robot tiles the LDS holds one sample
// of 6 waves per CU.
int adj_waves(int R, int n_items, int ncu) { return R == 2 ? 6 : (n_items <= ncu ? 8 : 4); }

size_t adj_lds(const DevCfg& c, int R, int KS, int W) { return (size_t)adj_fast_plan(c, R, KS, W).total * sizeof(float); }

}  // namespace

bool adjoint_fast_supported(const DevCfg& c) {
  if (c.D != 3 || c.n > 32 || c.m > 16 || c.H > 256) return false;
  return adj_lds(c, 2, 4, 6) <= kAdjLds;
}

hipError_t launch_adjoint_fast(const AdjFastArgs& a, const DevCfg* const* cfgs, int n_cfgs, int R, int KS, int ncu) {
  const int W = adj_waves(R, a.n_items, ncu);
  size_t lds = 0;
  for (int i = 0; i < n_cfgs; ++i) lds = std::max(lds, adj_lds(*cfgs[i], R, KS, W));
  switch (R * 100 + KS * 10 + W) {
    case 124: return launch(adjoint_fast_kernel<1, 2, 4>, a, 256, lds);
    case 128: return launch(adjoint_fast_kernel<1, 2, 8>, a, 512, lds);
    case 134: return launch(adjoint_fast_kernel<1, 3, 4>, a, 256, lds);
    case 138: return launch(adjoint_fast_kernel<1, 3, 8>, a, 512, lds);
    case 144: return launch(adjoint_fast_kernel<1, 4, 4>, a, 256, lds);
    case 148: return launch(adjoint_fast_kernel<1, 4, 8>, a, 512, lds);
    case 226: return launch(adjoint_fast_kernel<2, 2, 6>, a, 384, lds);
    case 236: return launch(adjoint_fast_kernel<2, 3, 6>, a, 384, lds);
    case 246: return launch(adjoint_fast_kernel<2, 4, 6>, a, 384, lds);
    default: return hipErrorNotSupported;
  }
}

hipError_t launch_adjoint_resid(const AdjFastArgs& a, const DevCfg* const* cfgs, int n_cfgs, int R, int KS) {
  size_t lds = 0;
  for (int i = 0; i < n_cfgs; ++i) lds = std::max(lds, adj_lds(*cfgs[i], R, KS, 4));
  switch (R * 10 + KS) {
    case 12: return launch(adjoint_resid_kernel<1, 2>, a, 256, lds);
    case 13: return launch(adjoint_resid_kernel<1, 3>, a, 256, lds);
    case 14: return launch(adjoint_resid_kernel<1, 4>, a, 256, lds);
    case 22: return launch(adjoint_resid_kernel<2, 2>, a, 256, lds);
    case 23: return launch(adjoint_resid_kernel<2, 3>, a, 256, lds);
    case 24: return launch(adjoint_resid_kernel<2, 4>, a, 256, lds);
    default: return hipErrorNotSupported;
  }
}

}  // namespace sf
