// MFMA fast path of the safety filter for 3D swarms (n <= 32 robots, degree <= 15, H <= 256).
//
// One workgroup (W = 2, 3 or 4 waves) owns one sample for the whole solve; xi, lambda and xi_bar
// stay in LDS.  The horizon is cut into 16-step time tiles and wave w owns tiles w, w + W, ...
// Per iteration (two workgroup barriers):
//   tiles (each wave, no barrier)
//     S1  Y_b = P_b xi for the bases (position, velocity, acceleration; eq. poly) as MFMA
//         products (fp32, or bf16/fp16 with hi/lo correction terms): rows = 16 times, columns =
//         16 robots of one axis; lane (col, grp) ends up holding robot col at times 4 grp + r.
//     S3  velocity/acceleration ball residuals in those registers (radial form of the d-step
//         with d in [0, 1]), skipped while a drift bound proves every ball inactive.
//     S2  collision residuals (alpha/beta/d steps in radial form): positions go to LDS; per
//         tile, a list of the pairs whose position boxes come within the safety distance plus a
//         margin, rebuilt only when some robot may have moved by more than the margin; the
//         listed pair-times are projected and scattered into an LDS accumulator.  A tile without
//         a residual is left out until some listed pair may have closed.
//     S4  g += P_b^T (rho_b R_b) as MFMA products, only for tiles with a nonzero residual; the
//         S1 output layout is exactly the A-operand layout this product needs.
//   barrier; tail (one wave per axis): multiplier step, and the structured QP step of eq. (xi_step) on the
//     free coefficients.
//   barrier
//
// The state is stored [axis][coefficient][16R robots], and lane (col, grp) of the S1 and S4 products and of the
// tail covers robot col and coefficients grp, grp + 4, ...: the S4 product, its basis operand's rows permuted
// (coef_of_row), leaves its result with the lanes that own it in the tail, so it is stored and summed without
// address arithmetic or bank conflicts.
//
// This header holds the kernels and their launchers; sf_fast_p<MP>_w<WS>[_r2].hip instantiate them per
// operand precision, workspace flag and robot tiles (so the instances compile in parallel, and the register
// allocation of one does not depend on the others: with the two-tile kernels in the same source the one-tile
// kernels spilled 19 registers), sf_fast.hip holds the host side (operand tables, plans, dispatch).
#pragma once

#include "sf_fast.h"

#include <cfloat>
#include <algorithm>
#include <cstring>

namespace sf {

void fast_set_error(const char* msg);

namespace fastk {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f4 mfma4(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// 16-bit operand types of v_mfma_f32_16x16x32_{bf16,f16}: MP = 1 bf16, MP = 2 fp16.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <int MP> struct Half;
template <> struct Half<1> { typedef __bf16 E; typedef bf16x8 V; };
template <> struct Half<2> { typedef _Float16 E; typedef f16x8 V; };

__device__ __forceinline__ f4 mfma16(bf16x8 a, bf16x8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ f4 mfma16(f16x8 a, f16x8 b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// B operands of the 16-bit S1 product for one robot tile and axis.  Lane (col, grp) covers
// coefficients 8 (grp & 1) .. + 7 of robot col.  First instruction: grp 0, 1 carry xi_hi against
// P_hi and grp 2, 3 carry xi_hi against P_lo; second instruction: grp 0, 1 carry xi_lo against
// P_hi, grp 2, 3 are zero.  The sum is P_hi xi_hi + P_lo xi_hi + P_hi xi_lo in fp32: the
// rounding residuals of both factors are fed back as correction terms.  x: coefficient 0 of the robot's row,
// `step` words apart.
template <int MP>
__device__ __forceinline__ void split_xi(const float* x, int step, bool real, int m, int grp,
                                         typename Half<MP>::V& b1, typename Half<MP>::V& b2) {
  typedef typename Half<MP>::E E;
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    const int k = 8 * (grp & 1) + v;
    const float xv = (real && k < m) ? x[k * step] : 0.0f;
    const E hi = static_cast<E>(xv);
    const E lo = static_cast<E>(xv - static_cast<float>(hi));
    b1[v] = hi;
    b2[v] = grp < 2 ? lo : static_cast<E>(0.0f);
  }
}

// Order LDS traffic between lanes of one wave (LDS instructions of a wave execute in order;
// this keeps the compiler from moving them and waits for outstanding LDS operations).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0));
}

// LDS plan (in 4-byte words).  Per-wave tile buffers: positions Xt and collision residual
// accumulator Ct as [axis][robot (16R)][time] with 16-word rows whose four 16-byte chunks are
// XOR-swizzled by the robot index (tile_at), so that the 16-byte accesses of 16 consecutive lanes
// hit distinct banks; boxes bb [robot][box_row(R)]; per tile, the list of pairs that can collide.  Once
// its time tiles are done, a wave reuses its own region for its partial back-projection (3 x 16R x 16
// words, as the products leave it) and, after the final residual pass, for its partial sums.
// Coefficient of row i of the S4 product's result: lane group i / 4 holds it in register i % 4.
__host__ __device__ constexpr int coef_of_row(int i) { return (i >> 2) + 4 * (i & 3); }
// Row strides (words) chosen so that the 16-byte accesses of 16 consecutive robots hit 16
// distinct groups of 4 banks (64 banks): boxes (lo xyz _, hi xyz _, pad) and 16-bit operands.  The
// forward kernel with two robot tiles keeps its boxes unpadded (two-way conflicts in the broad
// phase, which runs in rebuild iterations only) in the pair-list region, where the list of the tile
// being rebuilt and those after it are rewritten anyway, its pair lists in 16-bit entries, its pair
// table in each wave's pair-list region while that is free (set-up, final residual) and its 16-bit
// operand rows unpadded, with the 16-byte chunks permuted per row instead: an LDS plan that fits
// two workgroups of three or four waves per CU up to degree 12.
constexpr int kBoxRow = 12;
constexpr int kHBRow = 20;
__host__ __device__ constexpr int box_row(int R) { return R == 2 ? 8 : kBoxRow; }
__host__ __device__ constexpr int hb_row(int R) { return R == 2 ? 16 : kHBRow; }
// Index (16-bit units) of entry e of the 16-bit operand row `row` (axis * 16R + robot): e = kk for
// the hi part of coefficient kk, 16 + kk for its lo part.  Unpadded rows (two robot tiles) permute
// their four 16-byte chunks by bits 2-3 of the row, so the 16 rows of one lane group still fall in
// 16 distinct groups of 4 banks.
template <int R>
__device__ __forceinline__ int hb_at(int row, int e) {
  if constexpr (R == 2) return row * 32 + (e ^ (((row >> 2) & 3) << 3));
  else return row * (2 * kHBRow) + e;
}
// QP matrix row in LDS: the free coefficients of up to 4 KS in all, padded to whole 16-byte chunks.
__host__ __device__ constexpr int qp_row(int KS) { return (4 * KS - 6 + 3) & ~3; }
struct FastLds {
  int xi, lam, xb, xprev, pairs, mx, dxi, qp, hb, tiles, per_wave, total;
  int xt, ct, bb, plist, thr;   // offsets inside one wave's tile region
};
// Pair table and pair lists of a wave's tiles (count, then pair codes i | j << 8) per tile: 32-bit
// entries with one robot tile, 16-bit with two.
__host__ __device__ constexpr int plist_entries(int nr) { return nr * (nr - 1) / 2 + 1; }
template <int R> struct PairList { typedef int T; };
// Word offset, from the start of a wave's pair lists, of the boxes of its tile q with two robot tiles:
// the first 16-byte boundary after the 16-bit lists of tiles 0 .. q - 1.
__host__ __device__ constexpr int box_at(int q, int nr) { return (((q * plist_entries(nr) + 1) >> 1) + 3) & ~3; }
template <> struct PairList<2> { typedef uint16_t T; };

// What the instance (R, KS, MP) fixes comes first, so that most offsets are compile-time constants in the kernel; the
// state's stride depends on the degree (padded to 4 KS it would cost resident workgroups) and that of a wave's
// region on its number of time tiles.
__host__ __device__ inline FastLds fast_lds_plan(const DevCfg& c, int R, int KS, int W, int MP) {
  const int nr = 16 * R, Npmax = nr * (nr - 1) / 2, mfx = 4 * KS - 6;
  const int nst = 3 * c.m * nr;
  FastLds p;
  int o = 0;
  p.mx = o; o += 2 * 3 * nr;               // [evaluation parity][v, a, workspace][robot]: largest squares
  p.dxi = o; o += 4 * nr;                  // [robot]: max |change| of a free coefficient per axis, max |coefficient| over the iterates (bits)
  p.qp = o; o += 2 * mfx * qp_row(KS);     // X1, X01: rows of free coefficients, zero-padded
  p.hb = o; o += MP ? 3 * nr * hb_row(R) : 0; // 16-bit S1 B operands: [axis][robot][hi x16, lo x16 (, pad)]
  p.pairs = o; o += R == 2 ? 0 : Npmax;    // (two robot tiles: in the pair-list regions)
  // (two robot tiles: the previous iterate of the final residual lives in xi_out)
  p.xi = o; o += nst;                      // [axis][coefficient][16R robots], zero past the swarm
  p.lam = o; o += nst;
  p.xb = o; o += nst;                      // (two robot tiles: with the first-step correction for step 0)
  p.xprev = o; o += R == 1 ? nst : 0;      // first-step correction until step 0, the previous iterate from the last step
  o = (o + 3) & ~3;                        // 16-byte alignment of the tile buffers
  p.xt = 0;
  p.ct = 3 * nr * 16;
  // (two robot tiles: the boxes of tile q sit at the first 16-byte boundary after the pair lists of
  // tiles 0 .. q - 1, see box_at; those of the last tile run past the lists by at most 12 words)
  p.bb = R == 2 ? 0 : 6 * nr * 16;
  p.thr = R == 2 ? 6 * nr * 16 : p.bb + box_row(R) * nr;   // per tile of the wave, of at most 8 (see s_thr)
  p.plist = p.thr + 8;                     // per tile of the wave: [count, pairs...] kept across iterations
  const int NT = (c.H + 15) / 16, TQ = (NT + W - 1) / W;
  const int pw = p.plist + (R == 2 ? (TQ * plist_entries(nr) + 1) / 2 + 12 : TQ * plist_entries(nr));
  p.per_wave = (pw + 3) & ~3;
  p.tiles = o;
  o += W * p.per_wave;
  p.total = o;
  return p;
}

// Word offset of (row, t) in a tile buffer; row = axis * 16R + robot, t = 0..15.
__device__ __forceinline__ int tile_at(int row, int t) {
  return row * 16 + ((((t >> 2) ^ (row >> 2)) & 3) << 2) + (t & 3);
}

// Minimum / maximum over the four lanes col, col + 16, col + 32, col + 48 (every lane gets the
// result), with the row-swap instructions of gfx950 instead of LDS permutes.
__device__ __forceinline__ float grp_min(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fminf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fminf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float grp_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, false));
}

// Sum over aligned groups of NR (16 or 32) lanes; every lane of a group gets the same value
// (each step adds a lane's value and its partner's, and addition is commutative).
template <int NR>
__device__ __forceinline__ float group_sum(float v) {
  v = v + dpp<0xB1>(v);     // quad_perm [1, 0, 3, 2]
  v = v + dpp<0x4E>(v);     // quad_perm [2, 3, 0, 1]
  v = v + dpp<0x141>(v);    // row_half_mirror
  v = v + dpp<0x140>(v);    // row_mirror
  if constexpr (NR == 32) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  }
  return v;
}

// Maximum over aligned groups of NR (16 or 32) lanes; every lane of a group gets it.
template <int NR>
__device__ __forceinline__ float group_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  v = fmaxf(v, dpp<0x140>(v));
  if constexpr (NR == 32) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  }
  return v;
}

// Sum over the 64 lanes of a wave (all lanes active; every lane gets the same value).
__device__ __forceinline__ float wave_sum(float v) {
  v = group_sum<32>(v);
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// Maximum over the 64 lanes of a wave (all lanes active; every lane gets the result).
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  v = fmaxf(v, dpp<0x140>(v));
  return grp_max(v);
}

__device__ __forceinline__ void coll_resid3(float rx, float ry, float rz, float ia2, float ib2, float b,
                                            float& Rx, float& Ry, float& Rz) {
  const float ss = (rx * rx + ry * ry) * ia2 + rz * rz * ib2;
  if (ss >= FLT_MIN) {
    const float f = fminf(0.0f, 1.0f - rsqrtf(ss));
    Rx = f * rx;
    Ry = f * ry;
    Rz = f * rz;
  } else {   // coincident: atan2(0, 0) = 0 targets (0, 0, b) for the pair (lower, upper)
    Rx = 0.0f;
    Ry = 0.0f;
    Rz = -b;
  }
}

struct FastArgs {
  const DevCfg* cfgs;
  const float* tab;
  const uint4* a16;
  const DevProblem* probs;
  const WorkItem* items;
  int n_items;
  const float* xi_bar;
  const float* bvals;
  const float* xi0;
  const float* lam0;
  int iters;
  float* xi_out;
  float* lam_out;
  float* resid_out;
  int32_t* status_out;
  float* ckpt;
  int ckpt_every;
  int64_t ckpt_stride;
  int fpr;               // accumulate the fixed-point residual sum (resid_out is [S][3])
};

// Target waves per SIMD (the register budget): 3 with one robot tile (168 VGPRs; three waves per
// sample then keep four samples per CU resident); with two robot tiles 2 for three or four waves
// per sample (256 VGPRs; two workgroups per CU by LDS, six or eight waves) and 1 for two (the whole
// register file).
constexpr int waves_per_simd(int R, int MP, int W) { return R == 1 ? 3 : (W >= 3 ? 2 : 1); }
// Register budget, as waves per SIMD.  A CU takes four samples of three waves each.  At 168 registers they fill all
// twelve wave slots, and after a kernel with other workgroups the last sample often finds no slots of its shape, which
// costs another round: 16 robots x 1024 samples, 319 iterations, after a feasibility check took 1.75 ms against
// 1.22.  At 128 registers slots are left over: 1.24 ms in any order.  The 16-bit instances of up to 12 coefficients
// fit that with 5-12 spills, of which the iteration reloads one or two (11 in a workspace at two waves).  Those of 13
// to 16 do not: they spilled 66-95 registers, most of them inside the iteration (16 robots, degree 13, bf16, 100
// iterations: 1024 samples 1.76 ms at 128 registers, 0.85 at 168).  In fp32 124-155 registers are used as they come.
// The plans count waves_per_simd.
constexpr int reg_waves(int R, int KS, int MP, int W) {
  return R == 1 && MP != 0 && KS <= 3 ? 4 : waves_per_simd(R, MP, W);
}

// The whole solve of one work item (its samples) by one workgroup.  WPE: the register budget, as waves per SIMD.
// WS: the instance carries the workspace rows (evaluated for the configs that have them).
template <int R, int KS, int W, int MP, int WPE, int WS>
__device__ __forceinline__ void fast_item(const FastArgs& A, int it, float* smem) {
  const DevCfg* __restrict__ cfgs = A.cfgs;
  const float* __restrict__ tab = A.tab;
  const uint4* __restrict__ a16 = A.a16;
  const DevProblem* __restrict__ probs = A.probs;
  const WorkItem* __restrict__ items = A.items;
  const float* __restrict__ xi_bar = A.xi_bar;
  const float* __restrict__ bvals = A.bvals;
  const float* __restrict__ xi0 = A.xi0;
  const float* __restrict__ lam0 = A.lam0;
  const int iters = A.iters;
  float* __restrict__ xi_out = A.xi_out;
  float* __restrict__ lam_out = A.lam_out;
  float* __restrict__ resid_out = A.resid_out;
  int32_t* __restrict__ status_out = A.status_out;
  float* __restrict__ ckpt = A.ckpt;
  const int ckpt_every = A.ckpt_every;
  const int64_t ckpt_stride = A.ckpt_stride;
  const bool fpr = A.fpr != 0;
  const int rw = fpr ? 3 : 2;            // resid_out columns
  constexpr int NR = 16 * R;
  constexpr bool SLIM = WPE > 3;         // 128 registers: fewer operands held
  constexpr int PR = (NR * (NR - 1) / 2 + 63) / 64;   // 64-pair rounds of the broad phase
  // two robot tiles: no LDS copy of the previous iterate or of the first-step correction (see the plan)
  constexpr bool LEAN = R == 2;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nthr = 64 * W;
  {
    // per-lane indices from an opaque copy, so that the compiler keeps per-lane addresses next to
    // their uses instead of hoisting them to the kernel entry and spilling them
    int tid_i = threadIdx.x;
    asm volatile("" : "+v"(tid_i));
    const int tid = tid_i, lane = tid_i & 63;
    const int col = lane & 15, grp = lane >> 4;
    const WorkItem w = items[it];
    const DevProblem pr = probs[w.problem];
    const DevCfg c = cfgs[pr.cfg];
    const FastLds L = fast_lds_plan(c, R, KS, W, MP);
    const int n = c.n, m = c.m, mf = c.mf, H = c.H;
    const int nDm = n * 3 * m, nDf = n * 3 * mf, nRm = 3 * m * NR;
    const int Np = n * (n - 1) / 2;
    const int NT = (H + 15) / 16;
    const int TQ = (NT + W - 1) / W;            // time tiles per wave
    const float* X1 = tab + c.off_X1;
    const float* X01 = tab + c.off_X01;
    const float* Bmap = tab + c.off_Bmap;
    const float* Gfx = tab + c.off_Gfx;
    const float* Rfx = tab + c.off_Rfx;
    const float ia2 = (float)c.inv_a2, ib2 = (float)c.inv_b2, sb = (float)c.b;
    // workspace spheroid (eq. workspace_polar): centre, 1/a_w^2, 1/b_w^2, rho_w / rho_c
    const float wcx = c.ws_f[0], wcy = c.ws_f[1], wcz = c.ws_f[2];
    const float wia2 = c.ws_f[3], wib2 = c.ws_f[4], wsc = c.ws_f[5];
    const float vmax = (float)c.vmax, amax = (float)c.amax;
    const float n_rho_c = (float)c.n_rho_c, inv_n = 1.0f / (float)n;
    const float Lv = (float)c.lip_v, La = (float)c.lip_a;
    const float* bv = bvals + pr.bnd_off;
    float* sxi = smem + L.xi;
    float* slam = smem + L.lam;
    float* sxb = smem + L.xb;
    float* sxprev = smem + L.xprev;
    float* sdbar = smem + L.tiles;         // (set-up only)
    // pair table, lexicographic (i, j), i < j: shared with one robot tile; with two, each wave's copy
    // in its pair-list region, written where needed (set-up, final residual)
    typedef typename PairList<R>::T PT;
    PT* spairs = reinterpret_cast<PT*>(R == 2 ? smem + L.tiles + wave * L.per_wave + L.plist : smem + L.pairs);
    auto fill_pairs = [&](int t0, int stride) {
      for (int i = t0; i < n; i += stride) {
        int p = i * n - i * (i + 1) / 2;
        for (int j = i + 1; j < n; ++j) spairs[p++] = static_cast<PT>(i | (j << 8));
      }
    };
    // largest squares of the evaluated rows, as bits (non-negative floats order like their bits); the buffer
    // of one evaluation is read by the next iteration and cleared in its tail
    uint32_t* s_mx = reinterpret_cast<uint32_t*>(smem + L.mx);
    float* s_dxi = smem + L.dxi;
    // LDS word of element q of a sample ([robot][axis][coefficient]); the division by m <= 16 is exact for
    // the q < 1536 of a sample
    const unsigned minv = (65535u + m) / m;
    auto state_at = [&](int q) {
      const int row = (int)(((unsigned)q * minv) >> 16), robot = row / 3;
      return ((row - 3 * robot) * m + (q - row * m)) * NR + robot;
    };
    auto coef_at = [&](int robot, int d, int kk) { return (d * m + kk) * NR + robot; };
    // 16-bit hi/lo split of xi in the S1 B-operand layout, kept current by whoever writes xi
    typedef typename Half<MP == 0 ? 1 : MP>::E HE;
    HE* shb = reinterpret_cast<HE*>(smem + L.hb);
    auto put_split = [&](int robot, int d, int kk, float x) {
      const HE hi = static_cast<HE>(x);
      const HE lo = static_cast<HE>(x - static_cast<float>(hi));
      shb[hb_at<R>(d * NR + robot, kk)] = hi;
      shb[hb_at<R>(d * NR + robot, 16 + kk)] = lo;
    };
    float* wbuf = smem + L.tiles + wave * L.per_wave;
    // per tile of the wave: how far the summed drift may grow before some listed pair can collide
    float* s_thr = wbuf + L.thr;
    float* Xt = wbuf + L.xt;
    float* Ct = wbuf + L.ct;
    float* bb = wbuf + L.bb;
    // pinned coefficient r of a robot-axis row after the first step: Bmap (p0, v0, a0, pH, vH, aH)
    auto pinned = [&](int row, int r) {
      float acc = 0.0f;
      for (int s = 0; s < kNFix; ++s) acc = fmaf(Bmap[r * kNFix + s], bv[row * kNFix + s], acc);
      return acc;
    };
    auto fixed_k = [&](int r) { return r < 3 ? r : m - kNFix + r; };

    if constexpr (R == 2) fill_pairs(tid & 63, 64);
    else fill_pairs(tid, nthr);
    // QP matrices X1 (relative motion) and X01 (mean motion minus relative), [matrix][f][f2] (zero-padded)
    constexpr int QR = qp_row(KS), MFX = 4 * KS - 6;   // (MFX: free coefficients per robot-axis, at most)
    float* sX1 = smem + L.qp;
    for (int q = tid; q < 2 * MFX * QR; q += nthr) {
      const int f2 = q % QR, f = (q / QR) % MFX, mat = q / (QR * MFX);
      sX1[q] = f < mf && f2 < mf ? (mat == 0 ? X1 : X01)[f * mf + f2] : 0.0f;
    }
    for (int q = tid; q < nRm; q += nthr) sxi[q] = slam[q] = sxb[q] = 0.0f;   // (phantom robots stay zero)
    // basis operand tables: fp32 [tile][basis][S1 A operand, S4 B operand (x rho)][lane],
    // 16-bit [tile][basis][instruction][lane]
    const float4* a32c = reinterpret_cast<const float4*>(a16) + c.off_a32;
    const uint4* a16c = a16 + (MP == 1 ? c.off_a16[0] : c.off_a16[1]);
    __syncthreads();
    int mypair[PR];
#pragma unroll
    for (int r = 0; r < PR; ++r) mypair[r] = (64 * r + lane < Np) ? spairs[64 * r + lane] : -1;

    for (int sl = w.first; sl < w.first + w.count; ++sl) {
      // per-lane indices re-derived per sample from an opaque copy (see the iteration loop)
      int tid_s = threadIdx.x;
      asm volatile("" : "+v"(tid_s));
      const int tid = tid_s, lane = tid_s & 63;
      const int col = lane & 15, grp = lane >> 4;
      const int64_t coef = pr.coef_off + (int64_t)sl * nDm;
      const int64_t sidx = pr.sample_base + sl;
      for (int q = tid; q < nDm; q += nthr) {
        const float x = xi_bar[coef + q];
        const int e = state_at(q);
        sxb[e] = x;
        sxi[e] = xi0 ? xi0[coef + q] : x;
        slam[e] = lam0 ? lam0[coef + q] : 0.0f;
      }
      for (int q = tid; q < 4 * NR; q += nthr) s_dxi[q] = 0.0f;
      for (int q = tid; q < 2 * 3 * NR; q += nthr) s_mx[q] = 0u;
      for (int q = lane; q < 3 * NR * 16; q += 64) Ct[q] = 0.0f;
      // a sample the input check flagged (non-finite input) is not iterated; the status pass then
      // writes NaN over its outputs
      const int32_t in_flag = status_out ? __builtin_amdgcn_readfirstlane(status_out[sidx]) : 0;
      const int iters_s = in_flag < 0 ? 0 : iters;
      __syncthreads();
      // bound on |coefficient| over the iterates: the initial one and the pinned values
      for (int q = tid; q < 3 * n; q += nthr) {
        const int robot = q / 3, d = q - 3 * robot;
        float cmx = 0.0f;
        for (int kk = 0; kk < m; ++kk) cmx = fmaxf(cmx, fabsf(sxi[coef_at(robot, d, kk)]));
        for (int r = 0; r < kNFix; ++r) cmx = fmaxf(cmx, fabsf(pinned(q, r)));
        atomicMax(reinterpret_cast<uint32_t*>(s_dxi) + 4 * robot + 3, __float_as_uint(cmx));
      }
      if constexpr (MP != 0) {
        // one thread per (axis, robot, coefficient) of the padded operand rows (zeros outside)
        for (int q = tid; q < 3 * NR * 16; q += nthr) {
          const int row = q >> 4, kk = q & 15, d = row / NR, robot = row - d * NR;
          put_split(robot, d, kk, (robot < n && kk < m) ? sxi[coef_at(robot, d, kk)] : 0.0f);
        }
      }
      // the first QP step also moves the pinned coefficients (from xi0 to their boundary values);
      // its effect on the free ones is the correction G_rho (xi0 - xi_p) restricted to them
      for (int q = tid; q < 3 * kNFix; q += nthr) {
        const int d = q / kNFix, r = q - d * kNFix;
        float s = 0.0f;
        for (int i = 0; i < n; ++i) s += sxi[coef_at(i, d, fixed_k(r))] - pinned(i * 3 + d, r);
        sdbar[q] = s * inv_n;
      }
      __syncthreads();
      for (int q = tid; q < nDf; q += nthr) {
        const int row = q / mf, f = q - row * mf, robot = row / 3, d = row - 3 * robot;
        float acc = 0.0f;
        for (int r = 0; r < kNFix; ++r) {
          const float dl = sxi[coef_at(robot, d, fixed_k(r))] - pinned(row, r);
          acc = fmaf(n_rho_c * Gfx[f * kNFix + r], dl - sdbar[d * kNFix + r], acc);
          acc = fmaf(Rfx[f * kNFix + r], dl, acc);
        }
        if constexpr (LEAN) sxb[coef_at(robot, d, 3 + f)] += acc;   // step 0 reads xi_bar + correction
        else sxprev[coef_at(robot, d, 3 + f)] = acc;
      }
      __syncthreads();
      // bound-ball drift tracking, lane = robot, identical in every wave: margin to the bound at
      // the last evaluation and accumulated bound on the drift since then
      float mv = -1.0f, dv = 0.0f, ma = -1.0f, da = 0.0f;
      int prev_eval = 0;
      // the same for the workspace rows, as one slack: 1 - max ||M_w^{-1} (p - p_w)|| at the last
      // evaluation minus the scaled drift bounds of the positions since then
      float wsl = -1.0f;
      int ws_prev = 0;
      // pair lists: accumulated bound on the position change of robot `lane` per axis since the lists
      // were built (a position is a convex combination of its coefficients, so it moves by at most
      // the largest change of a coefficient)
      float px_ = 0.0f, py_ = 0.0f, pz_ = 0.0f;
      // this lane's share of the fixed-point residual sum_k ||xi^{k+1} - xi^k||^2 +
      // ||lambda^{k+1} - lambda^k||^2 (multiplier/QP-step lanes; lambda changes by -g)
      float fpsum = 0.0f;
      // summed bound on the change of any position (Euclidean) since the lists were built, and the rounding of a pair's
      // separation (both positions, at the evaluation and later; see the list margins)
      float drift = 0.0f, ptol = 0.0f;
      const float smin = (float)(c.a < c.b ? c.a : c.b);
      const float skx = (float)(c.skin * c.a) * 0.999f, skz = (float)(c.skin * c.b) * 0.999f;

      for (int k = 0; k < iters_s; ++k) {
        // Lane-dependent indices are re-derived from an opaque copy every iteration: otherwise the
        // compiler hoists every per-lane address of the loop body out of the sample loop and
        // spills them.
        int lane_o = tid;
        asm volatile("" : "+v"(lane_o));
        const int tid = lane_o, lane = lane_o & 63;
        const int col = lane & 15, grp = lane >> 4;
        if (ckpt && (k % ckpt_every) == 0) {
          const int64_t base = (int64_t)(k / ckpt_every) * 2 * ckpt_stride + coef;
          for (int q = tid; q < nDm; q += nthr) {
            const int e = state_at(q);
            ckpt[base + q] = sxi[e];
            ckpt[base + ckpt_stride + q] = slam[e];
          }
        }
        if ((resid_out || status_out) && k == iters_s - 1) {
          if constexpr (LEAN)   // overwritten with the result at the end (one robot tile: kept by the step)
            for (int q = tid; q < nDm; q += nthr) xi_out[coef + q] = sxi[state_at(q)];
        }
        // Velocity/acceleration at every grid time move by at most L * ||max_k |d xi_{i,d,k}| ||_2
        // per step (L = max_t sum_k |basis row|).  While the accumulated drift of every robot stays
        // below its margin to the bound at the last evaluation, the ball residuals are exactly zero
        // and S1/S3/S4 for that basis are skipped.  Iterations 0 and 1 always evaluate (the pinned
        // coefficients change in the first step).
        const int par = k & 1;
        const bool clear_mx = (prev_eval | ws_prev) != 0;   // the other buffer holds the last evaluation
        int eval_flags = 3;
        bool rebuild = true, ws_eval = false;
        float cmx;   // max |coefficient| of robot lane
        {
          // margins to the bounds measured by the previous iteration if it evaluated them
          // (every wave computes the same values).  The hardware square root (1 ulp) serves: the
          // test below keeps a 1e-4 relative slack, far above its error.  (Lanes past the swarm carry
          // other words and are left out of the tests.)
          const f4 dx = *reinterpret_cast<const f4*>(s_dxi + 4 * (lane & (NR - 1)));
          if ((prev_eval | ws_prev) != 0) {
            const uint32_t* pm = s_mx + (par ^ 1) * 3 * NR + (lane & (NR - 1));
            if (prev_eval & 1) {
              mv = vmax - __builtin_amdgcn_sqrtf(__uint_as_float(pm[0]));
              dv = 0.0f;
            }
            if (prev_eval & 2) {
              ma = amax - __builtin_amdgcn_sqrtf(__uint_as_float(pm[NR]));
              da = 0.0f;
            }
            if constexpr (WS)
              if (ws_prev) wsl = 1.0f - __builtin_amdgcn_sqrtf(__uint_as_float(pm[2 * NR]));
          }
          cmx = dx[3];
          const float dn = __builtin_amdgcn_sqrtf(dx[0] * dx[0] + dx[1] * dx[1] + dx[2] * dx[2]);
          px_ += dx[0];
          py_ += dx[1];
          pz_ += dx[2];
          drift = fmaf(drift, 1.8e-7f, drift + 1.0001f * group_max<NR>(dn));   // (rounded up: small steps count)
          dv += Lv * dn;
          da += La * dn;
          // ||M_w^{-1} (sum of steps)|| <= sum of ||M_w^{-1} step|| (triangle inequality)
          if constexpr (WS) wsl -= __builtin_amdgcn_sqrtf((dx[0] * dx[0] + dx[1] * dx[1]) * wia2 + dx[2] * dx[2] * wib2);
          const bool fv = c.vel_on && dv >= mv - 1e-4f * vmax;
          const bool fa = c.acc_on && da >= ma - 1e-4f * amax;
          // Workspace rows: a position moves per step by at most the largest coefficient change
          // per axis, so while max ||M_w^{-1} (p - p_w)|| at the last evaluation plus the summed
          // scaled drift stays below 1 (1e-4 slack) every workspace residual is exactly zero and the
          // rows are skipped.
          const bool fw = WS && c.ws_on && wsl <= 1e-4f;
          // Rebuild the pair lists when some robot may have moved by more than the margin they were
          // built with (and in iterations 0 and 1, where the pinned coefficients jump).
          const bool fr = px_ > skx || py_ > skx || pz_ > skz;
          if (k >= 2) {
            eval_flags = 0;
            rebuild = false;
            if (ballot(lane < n && (fv || fa || fw || fr)) != 0) {   // (most iterations evaluate nothing)
              eval_flags = (ballot(lane < n && fv) != 0 ? 1 : 0) | (ballot(lane < n && fa) != 0 ? 2 : 0);
              rebuild = ballot(lane < n && fr) != 0;
              if constexpr (WS) ws_eval = ballot(lane < n && fw) != 0;
            }
          } else if constexpr (WS) {
            ws_eval = c.ws_on;
          }
          if constexpr (WS) ws_prev = ws_eval;
        }
        prev_eval = eval_flags;
        if (rebuild) px_ = py_ = pz_ = drift = 0.0f;
        // Margins of the broad phase: twice the drift margin per axis, plus the rounding of the
        // positions.  A computed position is a rounded convex combination of its coefficients, off by
        // at most ~1.2e-5 of the largest |coefficient| (16-bit split products; fp32 far less); 2^-12
        // of a bound on that over the sample (running maximum, plus the most the coefficients can
        // grow before the next rebuild) holds for both robots of a pair in the build and every reuse
        // iteration.
        float mgx = 0.0f, mgz = 0.0f;
        if (rebuild) {
          const float tol = 2.44140625e-4f * (wave_max(cmx) + fmaxf(skx, skz));
          mgx = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(2.0f * skx + tol)));
          mgz = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(2.0f * skz + tol)));
          ptol = (MP == 0 ? 0.03125f : 0.5f) * tol;   // (four positions of up to 3e-7 or 1.2e-5 of the largest |coefficient|)
        }
        // Time tiles this wave evaluates.  After an evaluation that found no residual, the least ||s|| of the
        // tile's listed pairs (their separation in units of the safety distance) exceeds 1 by a margin, and a
        // pair closes by at most twice the drift of a position: until the drift since then reaches half the
        // margin, less the rounding, every residual of the tile is exactly zero and the tile is skipped.  Once
        // the early iterations have separated the robots, most tiles are: over 300 iterations a quarter of the tiles
        // is evaluated with 16 robots (1024 samples, bf16: 1.38 ms with every tile, 1.28 so), under half with 32 (4096
        // samples: 18.3 and 16.2 ms) and few with 8 robots x 4 samples (100 iterations, fp32: 340 and 296 us).
        unsigned need;
        {
          const bool force = rebuild || eval_flags != 0 || (WS && ws_eval);
          const int nq = wave < NT ? (NT - 1 - wave) / W + 1 : 0;
          const float th = s_thr[lane < TQ ? lane : 0];
          need = (unsigned)ballot(lane < nq && (force || drift > th));
        }
        // S1 B operand: xi^T, lane (col, grp) holds robot col, coefficient 4 s + grp
        float bx[MP == 0 ? R : 1][3][KS];
        // (two robot tiles at two waves per SIMD, and the workspace instances at 128 registers: the 16-bit
        // operands are re-read from LDS per product instead of held across the tiles, 48 or 24 registers fewer)
        constexpr bool HBR = R == 1 ? SLIM && WS != 0 : W >= 3;
        // (two robot tiles: offsets of this lane's hi and lo chunks from the first row of its robot
        // tile and axis, robot col, entries 8 (grp & 1) and 16 + 8 (grp & 1); see hb_at)
        const int hb_hi = hb_at<R>(col, 8 * (grp & 1)), hb_lo = hb_at<R>(col, 16 + 8 * (grp & 1));
        typename Half<MP == 0 ? 1 : MP>::V hb1[MP == 0 || HBR ? 1 : R][3], hb2[MP == 0 || HBR ? 1 : R][3];
        if constexpr (MP == 0) {
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
              for (int s = 0; s < KS; ++s) {
                // (past m the A operand is zero and the words read hold finite state)
                bx[rr][d][s] = sxi[(d * m + 4 * s + grp) * NR + 16 * rr + col];
              }
        } else if constexpr (!HBR) {
          // lane (col, grp) takes coefficients 8 (grp & 1) .. + 7 of robot col: hi in the first
          // instruction, lo in the second (see split_xi).  The second instruction's A operand is zero
          // for grp 2, 3, so their lo values (finite: the split of finite coefficients, zero past m)
          // add exact zeros and need no masking.
          typedef typename Half<MP == 0 ? 1 : MP>::V V;
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
              uint4 hi, lo;
              if constexpr (R == 1) {
                const uint4* hrow = reinterpret_cast<const uint4*>(shb + (d * NR + 16 * rr + col) * (2 * kHBRow));
                hi = hrow[grp & 1];
                lo = hrow[2 + (grp & 1)];
              } else {
                const HE* hrow = shb + (d * NR + 16 * rr) * (2 * hb_row(R));
                hi = *reinterpret_cast<const uint4*>(hrow + hb_hi);
                lo = *reinterpret_cast<const uint4*>(hrow + hb_lo);
              }
              hb1[rr][d] = __builtin_bit_cast(V, hi);
              hb2[rr][d] = __builtin_bit_cast(V, lo);   // (grp 2, 3 meet a zero A operand, see below)
            }
        }
        // S1 product for one basis of one tile: Y[rr][d] (lane (col, grp): robot col, times 4 grp + r)
        auto s1_32 = [&](const float4 av, f4 (&Y)[R][3]) {
          const float a1[4] = {av.x, av.y, av.z, av.w};
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int d = 0; d < 3; ++d) {
              f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
              for (int s = 0; s < KS; ++s) acc = mfma4(a1[s], bx[rr][d][s], acc);
              Y[rr][d] = acc;
            }
        };
        auto s1_16 = [&](const uint4 u1, const uint4 u2, f4 (&Y)[R][3]) {
          if constexpr (MP != 0) {
            typedef typename Half<MP>::V V;
            const V A1 = __builtin_bit_cast(V, u1);
            const V A2 = __builtin_bit_cast(V, u2);
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                if constexpr (HBR) {
                  const HE* hrow = shb + (d * NR + 16 * rr) * (2 * hb_row(R));
                  const uint4 lo = *reinterpret_cast<const uint4*>(hrow + hb_lo);
                  acc = mfma16(A1, __builtin_bit_cast(V, *reinterpret_cast<const uint4*>(hrow + hb_hi)), acc);
                  acc = mfma16(A2, __builtin_bit_cast(V, lo), acc);
                } else {
                  acc = mfma16(A1, hb1[rr][d], acc);
                  acc = mfma16(A2, hb2[rr][d], acc);
                }
                Y[rr][d] = acc;
              }
          }
        };
        f4 gacc[R][3];
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
          for (int d = 0; d < 3; ++d) gacc[rr][d] = f4{0.0f, 0.0f, 0.0f, 0.0f};
        float vm[2][R];           // max ||v||^2, ||a||^2 of robot col over this wave's tiles
        float wsm[WS ? R : 1];    // max ||M_w^{-1} (p - p_w)||^2 of robot col over this wave's tiles
#pragma unroll
        for (int rr = 0; rr < R; ++rr) vm[0][rr] = vm[1][rr] = 0.0f;
#pragma unroll
        for (int rr = 0; rr < (WS ? R : 1); ++rr) wsm[rr] = 0.0f;
        // position operands of the wave's first tile; each tile prefetches those of its next one
        float4 pa = {0.0f, 0.0f, 0.0f, 0.0f}, pb = {0.0f, 0.0f, 0.0f, 0.0f};
        uint4 pu1 = {0u, 0u, 0u, 0u}, pu2 = {0u, 0u, 0u, 0u};
        auto fetch = [&](int tau) {
          if constexpr (MP == 0) pa = a32c[((tau * 3) * 2) * 64 + lane];
          else {
            pu1 = a16c[((tau * 3) * 2) * 64 + lane];
            pu2 = a16c[((tau * 3) * 2 + 1) * 64 + lane];
          }
          pb = a32c[((tau * 3) * 2 + 1) * 64 + lane];
        };
        if (need != 0) fetch(wave + W * __builtin_ctz(need));

        // Issue priority (one robot tile): from the end of a wave's tiles through the partial write,
        // the barriers, the multiplier/QP step and the flags up to here, a wave runs at priority 2
        // (that work is serial for the sample: all its waves wait on it); in the tile phase the waves
        // with the most tiles (priority 1) carry the sample's longest path to the next barrier and
        // the others (0) have slack.  The SIMD issues from the waves of other
        // samples in that order, which shortens every sample's iteration.  (The two-tile kernels
        // gain about 1% from it and are left without.)
        if constexpr (R == 1) {
          if ((NT - 1 - wave) / W + 1 == TQ) __builtin_amdgcn_s_setprio(1);
          else __builtin_amdgcn_s_setprio(0);
        }
        while (need != 0) {
          const int q = __builtin_ctz(need);
          need &= need - 1;
          const int tau = wave + W * q;
          const int t0 = 16 * tau;
          const int nt = min(16, H - t0);
          const float4 ca = pa, cb = pb;
          const uint4 cu1 = pu1, cu2 = pu2;
          // narrow-phase lane mapping: lanes cover (pair, time) items, 64 / T pairs per round with
          // T = the tile's valid times rounded up to 4, 8 or 16.  A list kept from an earlier
          // iteration is read now (count and first round together), ahead of the products.
          typename PairList<R>::T* tl = reinterpret_cast<typename PairList<R>::T*>(wbuf + L.plist) + q * plist_entries(NR);
          // (two robot tiles: over the lists of this tile and the next, which a rebuild rewrites)
          float* const bbq = R == 2 ? wbuf + L.plist + box_at(q, NR) : bb;
          const int tsh = nt <= 4 ? 2 : (nt <= 8 ? 3 : 4);
          const int tt = lane & ((1 << tsh) - 1), ps = lane >> tsh, ppr = 64 >> tsh;
          const int kept_count = tl[0], kept_first = tl[1 + ps];
          if (need != 0) fetch(wave + W * __builtin_ctz(need));
          bool ws_nz = false;   // some workspace residual of the tile is nonzero (wave-uniform)
          // ---- S1 positions -> LDS, per-robot boxes over the tile in registers ----
          // (not needed when the tile's kept pair list is empty and no list or workspace row is
          // evaluated: then no residual of the tile is nonzero)
          if (rebuild || __builtin_amdgcn_readfirstlane(kept_count) > 0 || (WS && ws_eval)) {
            f4 Y[R][3];
            if constexpr (MP == 0) s1_32(ca, Y);
            else s1_16(cu1, cu2, Y);
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                *reinterpret_cast<f4*>(Xt + tile_at(d * NR + 16 * rr + col, 4 * grp)) = Y[rr][d];
              }
            // (rows past the horizon repeat the last grid time, so all 16 rows count)
#pragma unroll
            for (int rr = 0; rr < R && rebuild; ++rr) {
              float lo[3], hi[3];
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                const f4 v = Y[rr][d];
                lo[d] = grp_min(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])));
                hi[d] = grp_max(fmaxf(fmaxf(v[0], v[1]), fmaxf(v[2], v[3])));
              }
              if (grp == 0) {
                float* bq = bbq + (16 * rr + col) * box_row(R);
                *reinterpret_cast<f4*>(bq) = f4{lo[0], lo[1], lo[2], 0.0f};
                *reinterpret_cast<f4*>(bq + 4) = f4{hi[0], hi[1], hi[2], 0.0f};
              }
            }
            // workspace rows (F_w of eq. f_e) on the same positions: residual (p - p_w) max(0,
            // 1 - 1/||M_w^{-1} (p - p_w)||), scaled by rho_w / rho_c so that it joins the collision
            // residuals in the accumulator (zero until now) and their S4 product
            if (WS && ws_eval) {
              bool wnz = false;
#pragma unroll
              for (int rr = 0; rr < R; ++rr) {
                float mx = 0.0f;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const float qx = Y[rr][0][r] - wcx, qy = Y[rr][1][r] - wcy, qz = Y[rr][2][r] - wcz;
                  const float s2 = (qx * qx + qy * qy) * wia2 + qz * qz * wib2;
                  mx = fmaxf(mx, s2);
                  // (s2 > 1 is a normal number, so the bare hardware rsqrt serves)
                  const float f = (16 * rr + col < n && s2 > 1.0f) ? wsc * (1.0f - __builtin_amdgcn_rsqf(s2)) : 0.0f;
                  Y[rr][0][r] = f * qx;
                  Y[rr][1][r] = f * qy;
                  Y[rr][2][r] = f * qz;
                  wnz |= f != 0.0f;
                }
                wsm[WS ? rr : 0] = fmaxf(wsm[WS ? rr : 0], grp_max(mx));
              }
              if (ballot(wnz) != 0) {
                ws_nz = true;
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int d = 0; d < 3; ++d)
                    *reinterpret_cast<f4*>(Ct + tile_at(d * NR + 16 * rr + col, 4 * grp)) = Y[rr][d];
              }
            }
          }
          // ---- S1 velocity / acceleration, S3 bound balls in registers, S4 for nonzero tiles ----
#pragma unroll
          for (int b = 1; b < 3; ++b) {
            const bool on = b == 1 ? c.vel_on : c.acc_on;
            if (!on || !(eval_flags & b)) continue;
            const float lim = b == 1 ? vmax : amax;
            f4 Y[R][3];
            if constexpr (MP == 0) s1_32(a32c[((tau * 3 + b) * 2) * 64 + lane], Y);
            else s1_16(a16c[((tau * 3 + b) * 2) * 64 + lane], a16c[((tau * 3 + b) * 2 + 1) * 64 + lane], Y);
            bool nz = false;
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
              float mx = 0.0f;
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                const float vx = Y[rr][0][r], vy = Y[rr][1][r], vz = Y[rr][2][r];
                const float ss = vx * vx + vy * vy + vz * vz;
                mx = fmaxf(mx, ss);
                // (ss > lim^2 is a normal number, so the bare hardware rsqrt serves)
                const float f = ss > lim * lim ? 1.0f - lim * __builtin_amdgcn_rsqf(ss) : 0.0f;
                Y[rr][0][r] = f * vx;
                Y[rr][1][r] = f * vy;
                Y[rr][2][r] = f * vz;
                nz |= f != 0.0f;
              }
              vm[b - 1][rr] = fmaxf(vm[b - 1][rr], grp_max(mx));
            }
            if (ballot(nz) != 0) {
              const float4 bq = a32c[((tau * 3 + b) * 2 + 1) * 64 + lane];
              const float b4[4] = {bq.x, bq.y, bq.z, bq.w};
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int d = 0; d < 3; ++d)
#pragma unroll
                  for (int s = 0; s < 4; ++s) gacc[rr][d] = mfma4(b4[s], Y[rr][d][s], gacc[rr][d]);
            }
          }
          wave_sync();
          // ---- S2: broad phase over the tile (when the lists are rebuilt), narrow phase on the list ----
          // A pair is listed when its boxes, each gap shrunk by the margins above, are closer than the
          // safety distance (scaled, 1e-4 relative slack); until the next rebuild no unlisted pair can
          // come closer than the safety distance, so its residual is exactly zero.
          // (unused lanes test the pair (0, 1) and discard the result, so all box loads issue at once)
          int count = 0;
          int pnext = 0;
          if (rebuild) {
          bool act[PR];
#pragma unroll
          for (int r = 0; r < PR; ++r) {
            const int pij = mypair[r] >= 0 ? mypair[r] : (1 << 8);
            const int i = pij & 255, j = pij >> 8;
            const f4 li = *reinterpret_cast<const f4*>(bbq + i * box_row(R));
            const f4 hi = *reinterpret_cast<const f4*>(bbq + i * box_row(R) + 4);
            const f4 lj = *reinterpret_cast<const f4*>(bbq + j * box_row(R));
            const f4 hj = *reinterpret_cast<const f4*>(bbq + j * box_row(R) + 4);
            float g2 = 0.0f;
#pragma unroll
            for (int d = 0; d < 3; ++d) {
              const float gap = fmaxf(0.0f, fmaxf(lj[d] - hi[d], li[d] - hj[d]) - (d == 2 ? mgz : mgx));
              g2 += gap * gap * (d == 2 ? ib2 : ia2);
            }
            act[r] = mypair[r] >= 0 && g2 < 1.0001f;
            if (r % 2 == 1) __builtin_amdgcn_sched_barrier(0);   // box loads of two rounds in flight at most
          }
#pragma unroll
          for (int r = 0; r < PR; ++r) {
            const uint64_t mask = ballot(act[r]);
            if (act[r]) tl[1 + count + lanes_below(mask)] = mypair[r];
            count += __popcll(mask);
          }
          if (lane == 0) tl[0] = count;
          wave_sync();
          pnext = ps < count ? tl[1 + ps] : 0;
          } else {
            count = __builtin_amdgcn_readfirstlane(kept_count);
            pnext = ps < count ? kept_first : 0;
          }
          // narrow phase, one round of pairs per step; the next round's pair codes load meanwhile
          // (most tiles list at most one round)
          bool nzc = false;
          float near = FLT_MAX;   // least ||s||^2 of this lane's items
          for (int base = 0; base < count; base += ppr) {
            const int slot = base + ps;
            const int pij = pnext;
            pnext = slot + ppr < count ? tl[1 + slot + ppr] : 0;
            if (slot < count && tt < nt) {
              const int i = pij & 255, j = pij >> 8;
              const float rx = Xt[tile_at(0 * NR + i, tt)] - Xt[tile_at(0 * NR + j, tt)];
              const float ry = Xt[tile_at(1 * NR + i, tt)] - Xt[tile_at(1 * NR + j, tt)];
              const float rz = Xt[tile_at(2 * NR + i, tt)] - Xt[tile_at(2 * NR + j, tt)];
              float Rx, Ry, Rz;
              near = fminf(near, (rx * rx + ry * ry) * ia2 + rz * rz * ib2);
              coll_resid3(rx, ry, rz, ia2, ib2, sb, Rx, Ry, Rz);
              if (Rx != 0.0f || Ry != 0.0f || Rz != 0.0f) {
                nzc = true;
                atomicAdd(Ct + tile_at(0 * NR + i, tt), Rx);
                atomicAdd(Ct + tile_at(1 * NR + i, tt), Ry);
                atomicAdd(Ct + tile_at(2 * NR + i, tt), Rz);
                atomicAdd(Ct + tile_at(0 * NR + j, tt), -Rx);
                atomicAdd(Ct + tile_at(1 * NR + j, tt), -Ry);
                atomicAdd(Ct + tile_at(2 * NR + j, tt), -Rz);
              }
            }
          }
          const bool hit = ballot(nzc) != 0;
          {
            // (a tile without listed pairs needs no evaluation before the next rebuild)
            float th = hit ? -1.0f : FLT_MAX;
            if (!hit && count > 0)
              th = drift + 0.4999f * ((__builtin_amdgcn_sqrtf(-wave_max(-near)) - 1.0f) * smin - ptol);
            if (lane == 0) s_thr[q] = th;
          }
          if (ws_nz || hit) {
            wave_sync();
            const float b4[4] = {cb.x, cb.y, cb.z, cb.w};
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                f4* cp = reinterpret_cast<f4*>(Ct + tile_at(d * NR + 16 * rr + col, 4 * grp));
                const f4 cr = *cp;
                *cp = f4{0.0f, 0.0f, 0.0f, 0.0f};     // the accumulator is kept zero between tiles
#pragma unroll
                for (int s = 0; s < 4; ++s) gacc[rr][d] = mfma4(b4[s], cr[s], gacc[rr][d]);
              }
          }
          wave_sync();
        }
        if constexpr (R == 1) __builtin_amdgcn_s_setprio(2);   // (see the tile phase)
        // this wave's partial back-projection -> its own LDS region, as the products leave it (lane (col, grp),
        // register r: robot col, coefficient grp + 4 r), and its bound maxima
#pragma unroll
        for (int rr = 0; rr < R; ++rr)
#pragma unroll
          for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int r = 0; r < KS; ++r) wbuf[((d * R + rr) * KS + r) * 64 + lane] = gacc[rr][d][r];
        if ((eval_flags != 0 || (WS && ws_eval)) && grp == 0) {
#pragma unroll
          for (int rr = 0; rr < R; ++rr) {
            uint32_t* pm = s_mx + par * 3 * NR + 16 * rr + col;
            if (eval_flags & 1) atomicMax(pm, __float_as_uint(vm[0][rr]));
            if (eval_flags & 2) atomicMax(pm + NR, __float_as_uint(vm[1][rr]));
            if constexpr (WS)
              if (ws_eval) atomicMax(pm + 2 * NR, __float_as_uint(wsm[rr]));
          }
        }
        __syncthreads();
        if (clear_mx)
          for (int q = tid; q < 3 * NR; q += nthr) s_mx[(par ^ 1) * 3 * NR + q] = 0u;
        // Multiplier step and QP step of one axis per wave: lane (rb, q4) holds coefficients q4 + 4 r of robots
        // rb (and 16 + rb).  g = F^T rho R summed over the waves, lambda <- lambda - g,
        // y = xi_bar - xi + lambda - g (+ the first-step correction; with two robot tiles it sits in xi_bar) on the free coefficients, and
        // xi_free += X1 y + X01 mean_robots(y).  Every load is issued first and a scheduling barrier keeps the
        // arithmetic after them; y and its means then reach the lanes of a robot through LDS, in this axis'
        // partials of wave 0, which no other wave reads.  With two lanes per row, half the waves idle, the step was
        // a fifth of an iteration with one robot tile and a third with two (16 robots x 1024 samples, bf16, 300
        // iterations: 1.37 ms then and 1.32 so, every tile evaluated in both).
        for (int ax = wave; ax < 3; ax += W) {
          float* gp0 = smem + L.tiles + ax * (R * KS * 64);
          const int q4 = lane >> 4, rb = lane & 15;
          const int e0 = (ax * m + q4) * NR + rb;
          float xv[R][KS], lf[R][KS], xb[R][KS], gs[R][KS];
          // (two robot tiles or more than 12 coefficients: no registers left to load the matrices ahead; 16 robots of
          // degree 15, fp32, 100 iterations: 1024 samples 0.76 ms with 6-31 spills, 0.72 with the rows as they come)
          constexpr bool EARLY = R == 1 && KS <= 3;
          f4 x1[EARLY ? KS - 1 : 1][QR / 4], x01[EARLY ? KS - 1 : 1][QR / 4];
#pragma unroll
          for (int rr = 0; rr < R; ++rr)
#pragma unroll
            for (int r = 0; r < KS; ++r) {
              // (past m: other words, unused)
              const int e = e0 + 4 * r * NR + 16 * rr;
              xv[rr][r] = sxi[e];
              lf[rr][r] = slam[e];
              xb[rr][r] = sxb[e];
            }
          // (where the matrices are not loaded ahead the waves' partials come into registers of their own: the
          // compiler otherwise adds each as it comes, 18 to 24 LDS latencies in a row.  26 robots, degree 8, 39
          // samples, 150 iterations, bf16: 976 -> 922 us; with the matrices ahead it loads them together by itself)
          float part[EARLY ? 1 : W][R][KS];
          if constexpr (EARLY) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < KS; ++r) {
                gs[rr][r] = gp0[(rr * KS + r) * 64 + lane];
#pragma unroll
                for (int ww = 1; ww < W; ++ww) gs[rr][r] += gp0[ww * L.per_wave + (rr * KS + r) * 64 + lane];
              }
          } else {
#pragma unroll
            for (int ww = 0; ww < W; ++ww)
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int r = 0; r < KS; ++r) part[ww][rr][r] = gp0[ww * L.per_wave + (rr * KS + r) * 64 + lane];
          }
          const bool last = !LEAN && (resid_out || status_out) && k == iters_s - 1;
          auto qp_rows = [&](int r, f4 (&a)[QR / 4], f4 (&b)[QR / 4]) {   // (rows of a free coefficient, else any)
            const int fc = max(0, min(4 * r + q4 - 3, mf - 1));
#pragma unroll
            for (int cc = 0; cc < QR / 4; ++cc) {
              a[cc] = *reinterpret_cast<const f4*>(sX1 + fc * QR + 4 * cc);
              b[cc] = *reinterpret_cast<const f4*>(sX1 + (MFX + fc) * QR + 4 * cc);
            }
          };
#pragma unroll
          for (int r = 0; r < (EARLY ? KS - 1 : 0); ++r) qp_rows(r, x1[r], x01[r]);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (!EARLY) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < KS; ++r) {
                gs[rr][r] = part[0][rr][r];
#pragma unroll
                for (int ww = 1; ww < W; ++ww) gs[rr][r] += part[ww][rr][r];
              }
          }
          float* sy = gp0;                    // y [coefficient][16R robots], zero on the pinned ones
          float* sym = gp0 + L.per_wave;      // robot means [coefficient][16]
          float sum[KS];
#pragma unroll
          for (int r = 0; r < KS; ++r) {
            const int kk = 4 * r + q4;
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
              const float g = gs[rr][r];
              lf[rr][r] -= g;
              float yv = xb[rr][r] - xv[rr][r] + lf[rr][r] - g;
              if constexpr (!LEAN)
                if (k == 0 && kk >= 3 && kk < m - 3) yv += sxprev[e0 + 4 * r * NR + 16 * rr];
              const float y = (kk >= 3 && kk < m - 3 && 16 * rr + rb < n) ? yv : 0.0f;
              sy[kk * NR + 16 * rr + rb] = y;
              const float t = group_sum<16>(y);
              sum[r] = rr == 0 ? t : sum[r] + t;
            }
          }
#pragma unroll
          for (int r = 0; r < KS; ++r) sym[(4 * r + q4) * 16 + rb] = sum[r] * inv_n;
          wave_sync();
          float ya[R][MFX], yba[MFX];
#pragma unroll
          for (int f2 = 0; f2 < MFX; ++f2) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr) ya[rr][f2] = sy[(f2 + 3) * NR + 16 * rr + rb];
            yba[f2] = sym[(f2 + 3) * 16];
          }
          float acc[R][KS];
          auto qp_step = [&](int r, const f4 (&a)[QR / 4], const f4 (&b)[QR / 4]) {
#pragma unroll
            for (int f2 = 0; f2 < MFX; ++f2)
#pragma unroll
              for (int rr = 0; rr < R; ++rr) {
                acc[rr][r] = fmaf(a[f2 / 4][f2 % 4], ya[rr][f2], acc[rr][r]);
                acc[rr][r] = fmaf(b[f2 / 4][f2 % 4], yba[f2], acc[rr][r]);
              }
          };
          float dmax[R], cmax[R];
          // new coefficients 4 r + q4 (phantom robots store their zeros)
          auto finish = [&](int r) {
            const int kk = 4 * r + q4;
#pragma unroll
            for (int rr = 0; rr < R; ++rr) {
              const bool upd = kk >= 3 && kk < m - 3 && 16 * rr + rb < n;
              if (fpr && 16 * rr + rb < n && kk < m) {
                fpsum = fmaf(gs[rr][r], gs[rr][r], fpsum);
                if (upd) fpsum = fmaf(acc[rr][r], acc[rr][r], fpsum);
              }
              dmax[rr] = fmaxf(dmax[rr], upd ? fabsf(acc[rr][r]) : 0.0f);
              xb[rr][r] = upd ? xv[rr][r] + acc[rr][r] : xv[rr][r];
              cmax[rr] = fmaxf(cmax[rr], kk < m ? fabsf(xb[rr][r]) : 0.0f);
            }
            if (kk < m) {
#pragma unroll
              for (int rr = 0; rr < R; ++rr) {
                const int e = e0 + 4 * r * NR + 16 * rr;
                sxi[e] = xb[rr][r];
                slam[e] = lf[rr][r];
                if constexpr (!LEAN)
                  if (last) sxprev[e] = xv[rr][r];
                if constexpr (MP != 0) put_split(16 * rr + rb, ax, kk, xb[rr][r]);
              }
            }
          };
#pragma unroll
          for (int rr = 0; rr < R; ++rr) dmax[rr] = cmax[rr] = 0.0f;
#pragma unroll
          for (int r = 0; r < KS; ++r)
#pragma unroll
            for (int rr = 0; rr < R; ++rr) acc[rr][r] = 0.0f;
#pragma unroll
          for (int r = 0; r < KS - 1; ++r) {
            if constexpr (!EARLY) qp_rows(r, x1[0], x01[0]);
            qp_step(r, x1[EARLY ? r : 0], x01[EARLY ? r : 0]);
            if constexpr (!EARLY) finish(r);
          }
          if (m == 4 * KS) {   // (else the last coefficients of every lane are pinned)
            f4 xl[QR / 4], xl01[QR / 4];
            qp_rows(KS - 1, xl, xl01);
            qp_step(KS - 1, xl, xl01);
          }
#pragma unroll
          for (int r = EARLY ? 0 : KS - 1; r < KS; ++r) finish(r);
#pragma unroll
          for (int rr = 0; rr < R; ++rr) {
            const float dm = grp_max(dmax[rr]);
            if (q4 == 0) s_dxi[4 * (16 * rr + rb) + ax] = dm;
            atomicMax(reinterpret_cast<uint32_t*>(s_dxi) + 4 * (16 * rr + rb) + 3, __float_as_uint(cmax[rr]));
          }
          if (k == 0) {
            // the pinned coefficients move to their boundary values in the first step, and with two robot tiles
            // xi_bar drops the correction again
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int r = 0; r < KS; ++r) {
                const int kk = 4 * r + q4, robot = 16 * rr + rb, e = e0 + 4 * r * NR + 16 * rr;
                if (robot < n && kk < m) {
                  const int row = robot * 3 + ax;
                  if (kk >= 3 && kk < m - 3) {
                    if constexpr (LEAN) sxb[e] = xi_bar[coef + row * m + kk];
                  } else {
                    const float xp = pinned(row, kk < 3 ? kk : kk - (m - kNFix));
                    if (fpr) fpsum = fmaf(xp - xv[rr][r], xp - xv[rr][r], fpsum);
                    sxi[e] = xp;
                    if constexpr (MP != 0) put_split(robot, ax, kk, xp);
                  }
                }
              }
          }
          if constexpr (W >= 3) break;   // (one axis per wave)
        }
        __syncthreads();
      }

      // ---- primal residual of the last step (dense over pairs) ----
      // Bound by the latency of its chains: operand splits, products, pair rounds.  The operands of both iterates
      // are formed once where the registers hold them, each tile's basis operands load together and the pair rounds go
      // two at a time (13 robots in a workspace, 333 samples, 60 iterations, fp16: 268 us for the whole solve, 3% more
      // with the operands formed per product).
      float rmax = 0.0f;   // its largest block norm (thread 0)
      if (resid_out || status_out) {
        float ss = 0.0f, mx = 0.0f;
        if (iters_s > 0) {
          // (lane index from an opaque copy, so that nothing is computed ahead of the iterations)
          int ln = threadIdx.x & 63;
          asm volatile("" : "+v"(ln));
          const int lane = ln, col = ln & 15, grp = ln >> 4;
          if constexpr (R == 2) {   // the wave's pair lists are no longer needed
            fill_pairs(lane, 64);
            wave_sync();
          }
          // B operands of the basis products for the previous and the new iterate, formed once for all tiles
          // (previous: in LDS or, with two robot tiles, in xi_out; at 128 registers and with two tiles in fp32 the
          // new one is read per product, which keeps the registers within the budget)
          constexpr int HELD = SLIM || (R == 2 && MP == 0) ? 1 : 2;
          typedef typename Half<MP == 0 ? 1 : MP>::V V;
          float b32[HELD][MP == 0 ? R : 1][3][KS];
          V b16[HELD][MP == 0 ? 1 : R][3][2];
#pragma unroll
          for (int it = 0; it < HELD; ++it) {
            const float* src = it == 0 ? (LEAN ? xi_out + coef : sxprev) : sxi;
            const bool glob = LEAN && it == 0;
            const int sr = glob ? 3 * m : 1, sd = glob ? m : m * NR, sk = glob ? 1 : NR;
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                const int robot = 16 * rr + col;
                if constexpr (MP == 0) {
#pragma unroll
                  for (int s = 0; s < KS; ++s) {
                    const int kk = 4 * s + grp;
                    b32[it][rr][d][s] = (robot < n && kk < m) ? src[robot * sr + d * sd + kk * sk] : 0.0f;
                  }
                } else {
                  split_xi<MP>(src + (robot < n ? robot * sr + d * sd : 0), sk, robot < n, m, grp, b16[it][rr][d][0],
                               b16[it][rr][d][1]);
                }
              }
          }
          // one basis product of a tile for an iterate
          auto prod = [&](int it, const uint4 (&au)[2], f4 (&Y)[R][3]) __attribute__((always_inline)) {
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
              for (int d = 0; d < 3; ++d) {
                f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                if constexpr (MP == 0) {
                  const f4 a1 = __builtin_bit_cast(f4, au[0]);
#pragma unroll
                  for (int s = 0; s < KS; ++s) {
                    // (past m the A operand is zero and the words read hold finite state, as do phantom robots)
                    const float v = it < HELD ? b32[it < HELD ? it : 0][rr][d][s]
                                              : sxi[(d * m + 4 * s + grp) * NR + 16 * rr + col];
                    acc = mfma4(a1[s], v, acc);
                  }
                } else {
                  V hi, lo;
                  if (it < HELD) {
                    hi = b16[it < HELD ? it : 0][rr][d][0];
                    lo = b16[it < HELD ? it : 0][rr][d][1];
                  } else {
                    const HE* hrow = shb + (d * NR + 16 * rr) * (2 * hb_row(R));
                    hi = __builtin_bit_cast(V, *reinterpret_cast<const uint4*>(hrow + hb_at<R>(col, 8 * (grp & 1))));
                    lo = __builtin_bit_cast(V, *reinterpret_cast<const uint4*>(hrow + hb_at<R>(col, 16 + 8 * (grp & 1))));
                  }
                  acc = mfma16(__builtin_bit_cast(V, au[0]), hi, acc);
                  acc = mfma16(__builtin_bit_cast(V, au[1]), lo, acc);
                }
                Y[rr][d] = acc;
              }
          };
#pragma unroll 1
          for (int q = 0; q < TQ; ++q) {
            const int tau = wave + W * q;
            if (tau >= NT) break;
            const int t0 = 16 * tau;
            const int nt = min(16, H - t0);
            uint4 au[3][2];
#pragma unroll
            for (int b = 0; b < 3; ++b) {
              if constexpr (MP == 0) {
                au[b][0] = __builtin_bit_cast(uint4, a32c[((tau * 3 + b) * 2) * 64 + lane]);
              } else {
                au[b][0] = a16c[((tau * 3 + b) * 2) * 64 + lane];
                au[b][1] = a16c[((tau * 3 + b) * 2 + 1) * 64 + lane];
              }
            }
#pragma unroll
            for (int b = 0; b < 3; ++b) {
              if (b > 0 && !(b == 1 ? c.vel_on : c.acc_on)) continue;
              const float lim = b == 1 ? vmax : amax;
              f4 Y[R][3];
              prod(0, au[b], Y);
              if (b == 0) {
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int d = 0; d < 3; ++d)
                    *reinterpret_cast<f4*>(Xt + tile_at(d * NR + 16 * rr + col, 4 * grp)) = Y[rr][d];
              } else {
                // targets of the bound balls at the previous iterate: e = v - R(v)
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int r = 0; r < 4; ++r) {
                    const float vx = Y[rr][0][r], vy = Y[rr][1][r], vz = Y[rr][2][r];
                    const float s2 = vx * vx + vy * vy + vz * vz;
                    const float f = s2 > lim * lim ? 1.0f - lim * rsqrtf(s2) : 0.0f;
                    Y[rr][0][r] = vx - f * vx;
                    Y[rr][1][r] = vy - f * vy;
                    Y[rr][2][r] = vz - f * vz;
                  }
              }
              f4 Yn[R][3];
              prod(1, au[b], Yn);
              if (b == 0) {
#pragma unroll
                for (int rr = 0; rr < R; ++rr)
#pragma unroll
                  for (int d = 0; d < 3; ++d)
                    *reinterpret_cast<f4*>(Ct + tile_at(d * NR + 16 * rr + col, 4 * grp)) = Yn[rr][d];
                if (WS && c.ws_on) {
                  // workspace rows: r_p = p_new - e(p_prev), e = p - (p - p_w) max(0, 1 - 1/||s||)
#pragma unroll
                  for (int rr = 0; rr < R; ++rr)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                      const float qx = Y[rr][0][r] - wcx, qy = Y[rr][1][r] - wcy, qz = Y[rr][2][r] - wcz;
                      const float s2 = (qx * qx + qy * qy) * wia2 + qz * qz * wib2;
                      const float f = s2 > 1.0f ? 1.0f - rsqrtf(s2) : 0.0f;
                      const float px = Yn[rr][0][r] - (Y[rr][0][r] - f * qx);
                      const float py = Yn[rr][1][r] - (Y[rr][1][r] - f * qy);
                      const float pz = Yn[rr][2][r] - (Y[rr][2][r] - f * qz);
                      const bool real = 4 * grp + r < nt && 16 * rr + col < n;   // grid times, robots
                      const float nrm = real ? px * px + py * py + pz * pz : 0.0f;
                      ss += nrm;
                      mx = fmaxf(mx, nrm);
                    }
                }
                continue;
              }
              // bound balls: r_p = v_new - e(v_prev)
#pragma unroll
              for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const float px = Yn[rr][0][r] - Y[rr][0][r];
                  const float py = Yn[rr][1][r] - Y[rr][1][r];
                  const float pz = Yn[rr][2][r] - Y[rr][2][r];
                  const float nrm = 4 * grp + r < nt ? px * px + py * py + pz * pz : 0.0f;   // grid times only
                  ss += nrm;
                  mx = fmaxf(mx, nrm);
                }
            }
            wave_sync();
            // four pairs of up to 16 times per round, two rounds in flight and the codes of the next two loading
            // meanwhile; a lane adds its pairs in order.
            int next[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) next[u] = spairs[max(0, min(4 * u + grp, Np - 1))];
            for (int base = 0; base < Np; base += 8) {
              float nrm[2];
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const int pij = next[u];
                const int i = pij & 255, j = pij >> 8;
                next[u] = spairs[min(base + 8 + 4 * u + grp, Np - 1)];
                float rp[3], rn[3];
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                  rp[d] = Xt[tile_at(d * NR + i, col)] - Xt[tile_at(d * NR + j, col)];
                  rn[d] = Ct[tile_at(d * NR + i, col)] - Ct[tile_at(d * NR + j, col)];
                }
                float Rx, Ry, Rz;
                coll_resid3(rp[0], rp[1], rp[2], ia2, ib2, sb, Rx, Ry, Rz);
                const float px = rn[0] - (rp[0] - Rx), py = rn[1] - (rp[1] - Ry), pz = rn[2] - (rp[2] - Rz);
                nrm[u] = px * px + py * py + pz * pz;
              }
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const float v = base + 4 * u + grp < Np && col < nt ? nrm[u] : 0.0f;
                ss += v;
                mx = fmaxf(mx, v);
              }
            }
            wave_sync();
          }
        }
        // per-wave sums and maxima (cross-lane, in a fixed order) in the wave's own region, then
        // combined in wave order
        {
          const float ws = wave_sum(ss), wm = wave_max(mx), wf = wave_sum(fpsum);
          if (lane == 0) {
            wbuf[0] = ws;
            wbuf[1] = wm;
            wbuf[2] = wf;
          }
        }
        __syncthreads();
        if (tid == 0) {
          float s = 0.0f, mm = 0.0f, fs = 0.0f;
          for (int ww = 0; ww < W; ++ww) {
            const float* pw = smem + L.tiles + ww * L.per_wave;
            s += pw[0];
            mm = fmaxf(mm, pw[1]);
            fs += pw[2];
          }
          rmax = sqrtf(mm);
          if (resid_out) {
            resid_out[sidx * rw + 0] = s;
            resid_out[sidx * rw + 1] = rmax;
            if (fpr) resid_out[sidx * rw + 2] = fs;
          }
        }
        __syncthreads();
      }
      for (int q = tid; q < nDm; q += nthr) {
        const int e = state_at(q);
        xi_out[coef + q] = sxi[e];
        if (lam_out) lam_out[coef + q] = slam[e];
      }
      // convergence bits (the status pass adds the finiteness of the outputs)
      if (status_out && tid == 0) status_out[sidx] = in_flag < 0 ? in_flag : sample_status<float>(false, false, rmax, iters_s);
      __syncthreads();
    }
  }
}

// One workgroup per work item (grid-stride), single shape class.
template <int R, int KS, int W, int MP, int WPE, int WS>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
fast_project_kernel(FastArgs A) {
  extern __shared__ __align__(16) float smem[];
  for (int it = blockIdx.x; it < A.n_items; it += gridDim.x) fast_item<R, KS, W, MP, WPE, WS>(A, it, smem);
}

// Recomputes several checkpoint segments at once for the reverse mode: workgroup (segment, work item) runs
// the segment's iterations from its checkpoint (xi0, lam0: that of the first segment, seg_in elements apart)
// and writes the state of every iteration (ckpt: those of the first segment, seg_out apart), the last one
// after them.  A segment has few iterations, so one launch per segment leaves the chip waiting for each
// sample's set-up: 16 robots x 512 samples, ten segments of ten iterations, 70 us each, 440 us together.
template <int R, int KS, int W, int MP, int WPE, int WS>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
fast_segments_kernel(FastArgs A, int nseg, int64_t seg_in, int64_t seg_out, int iters_total) {
  extern __shared__ __align__(16) float smem[];
  for (int it = blockIdx.x; it < A.n_items * nseg; it += gridDim.x) {
    const int seg = it / A.n_items;
    FastArgs B = A;
    B.iters = min(A.iters, iters_total - seg * A.iters);
    B.xi0 += seg * seg_in;
    B.lam0 += seg * seg_in;
    B.ckpt += seg * seg_out;
    B.xi_out = B.ckpt + B.iters * 2 * A.ckpt_stride;
    B.lam_out = B.xi_out + A.ckpt_stride;
    fast_item<R, KS, W, MP, WPE, WS>(B, it - seg * A.n_items, smem);
  }
}

// Persistent kernel over the work items of one robot-tile class (R tiles of 16 robots) of a
// ragged batch: workgroups pull items (sorted by decreasing cost on the host) from an atomic
// queue until it is empty.  Every wave reaches the exit once the queue is drained.
template <int R, int KS, int W, int MP, int WPE, int WS>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
fast_batched_kernel(FastArgs A, int* __restrict__ queue) {
  extern __shared__ __align__(16) float smem[];
  __shared__ int next;
  for (;;) {
    if (threadIdx.x == 0) next = atomicAdd(queue, 1);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(next);
    __syncthreads();
    if (it >= A.n_items) break;
    fast_item<R, KS, W, MP, WPE, WS>(A, it, smem);
  }
}

// Kernel instances: R robot tiles of 16, KS k-steps of 4 coefficients, W waves per workgroup.
FastArgs make_fast_args(const LaunchArgs& a, const float* tab32, const uint4* a16) {
  FastArgs f;
  f.cfgs = a.cfgs; f.tab = tab32; f.a16 = a16; f.probs = a.probs; f.items = a.items; f.n_items = a.n_items;
  f.xi_bar = static_cast<const float*>(a.xi_bar); f.bvals = static_cast<const float*>(a.bvals);
  f.xi0 = static_cast<const float*>(a.xi0); f.lam0 = static_cast<const float*>(a.lam0); f.iters = a.iters;
  f.xi_out = static_cast<float*>(a.xi_out); f.lam_out = static_cast<float*>(a.lam_out);
  f.resid_out = static_cast<float*>(a.resid_out); f.status_out = a.status_out; f.ckpt = static_cast<float*>(a.ckpt);
  f.ckpt_every = a.ckpt_every; f.ckpt_stride = a.ckpt_stride;
  f.fpr = (a.flags & SF_FP_RESIDUAL) != 0;
  return f;
}

template <int R, int KS, int W, int MP, int WS, int WPE>
hipError_t launch_instance(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16) {
  auto kern = fast_project_kernel<R, KS, W, MP, WPE, WS>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds_bytes[W - 2][MP]);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(a.n_items), dim3(64 * W), p.lds_bytes[W - 2][MP], a.stream, make_fast_args(a, tab32, a16));
  return hipGetLastError();
}

// The instance of a launch.  At 128 registers the workspace instances re-read their operands per product, which costs
// 4-5% (13 robots, degree 9, 333 samples, 60 iterations, fp16: 279 us, 268 with the operands held in 168) and pays
// only where the wave slots of 168 registers are all taken (see reg_waves): batches that leave some free hold them
// (1024 samples of 16 robots, 300 iterations, bf16, after a feasibility check: 1.37 ms against 1.41; 3000 samples,
// 100 iterations: 1.56 against 1.66).  Without a workspace the operands are held in either budget.
template <int R, int KS, int W, int MP, int WS>
hipError_t launch_sized(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16) {
  constexpr int kFull = waves_per_simd(R, MP, W), kBudget = reg_waves(R, KS, MP, W);
  if constexpr (WS != 0 && kBudget != kFull)
    if ((int64_t)a.n_items * W < (int64_t)4 * kFull * p.ncu)
      return launch_instance<R, KS, W, MP, WS, kFull>(p, a, tab32, a16);
  return launch_instance<R, KS, W, MP, WS, kBudget>(p, a, tab32, a16);
}


template <int R, int KS, int W, int MP, int WS>
hipError_t launch_segments_instance(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16) {
  auto kern = fast_segments_kernel<R, KS, W, MP, reg_waves(R, KS, MP, W), WS>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds_bytes[W - 2][MP]);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)(a.n_items * a.nseg)), dim3(64 * W), p.lds_bytes[W - 2][MP], a.stream,
                     make_fast_args(a, tab32, a16), a.nseg, a.seg_in, a.seg_out, a.iters_total);
  return hipGetLastError();
}

// Single-shape batch, at the waves per sample a small batch runs with (4, with a workspace 3).
template <int MP, int WS, int R>
hipError_t launch_segments_mp(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16) {
  constexpr int W = WS ? 3 : 4;
  switch (p.KS) {
    case 2: return launch_segments_instance<R, 2, W, MP, WS>(p, a, tab32, a16);
    case 3: return launch_segments_instance<R, 3, W, MP, WS>(p, a, tab32, a16);
    case 4: return launch_segments_instance<R, 4, W, MP, WS>(p, a, tab32, a16);
    default: break;
  }
  fast_set_error("no kernel instance for this shape");
  return hipErrorNotSupported;
}

template <int R, int KS, int W, int MP, int WS>
hipError_t launch_class(const FastClass& C, const FastArgs& f, int grid, int* queue, hipStream_t stream) {
  // (a persistent launch loses nothing when a workgroup finds no slots, the others take its items, so the workspace
  // instances hold their operands: 700 samples of 16 and 12 robots, 100 iterations, bf16: 902 -> 858 us)
  constexpr int kBudget = WS != 0 ? waves_per_simd(R, MP, W) : reg_waves(R, KS, MP, W);
  auto kern = fast_batched_kernel<R, KS, W, MP, kBudget, WS>;
  const size_t lds = C.lds_bytes[W - 2][MP];
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * W), lds, stream, f, queue);
  return hipGetLastError();
}

// One class of a persistent launch sequence with W waves per workgroup; grid > 0: workgroups (at most
// the class's work items), 0: the class's default.
template <int R, int KS, int MP, int WS>
hipError_t launch_class_w(const FastClass& C, const FastArgs& f, int grid, int W, int* queue, hipStream_t stream) {
  switch (W) {
    case 2: return launch_class<R, KS, 2, MP, WS>(C, f, grid, queue, stream);
    case 3: return launch_class<R, KS, 3, MP, WS>(C, f, grid, queue, stream);
    case 4:
      if constexpr (WS == 0) return launch_class<R, KS, 4, MP, WS>(C, f, grid, queue, stream);
      break;
    default: break;
  }
  fast_set_error("no persistent kernel instance for this shape");
  return hipErrorNotSupported;
}

// Single-shape launch of the instance for (R, KS, W) of this precision and workspace flag.
template <int MP, int WS, int R, int KS>
hipError_t launch_single_w(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int W) {
  switch (W) {
    case 2: return launch_sized<R, KS, 2, MP, WS>(p, a, tab32, a16);
    case 3: return launch_sized<R, KS, 3, MP, WS>(p, a, tab32, a16);
    case 4:   // (with the workspace rows: 2 or 3 waves per workgroup)
      if constexpr (WS == 0) return launch_sized<R, KS, 4, MP, WS>(p, a, tab32, a16);
      break;
    default: break;
  }
  fast_set_error("no kernel instance for this shape");
  return hipErrorNotSupported;
}
template <int MP, int WS, int R>
hipError_t launch_single_mp(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int W) {
  switch (p.KS) {
    case 2: return launch_single_w<MP, WS, R, 2>(p, a, tab32, a16, W);
    case 3: return launch_single_w<MP, WS, R, 3>(p, a, tab32, a16, W);
    case 4: return launch_single_w<MP, WS, R, 4>(p, a, tab32, a16, W);
    default: break;
  }
  fast_set_error("no kernel instance for this shape");
  return hipErrorNotSupported;
}

// Class ci (of R robot tiles) of a persistent launch sequence with W waves per workgroup; grid > 0: workgroups
// (at most the class's work items), 0: the class's default.
template <int MP, int WS, int R>
hipError_t launch_batched_mp(const FastPlan& p, const LaunchArgs& a, const float* tab32, const uint4* a16, int ci,
                             int grid, int W) {
  const FastClass& C = p.cls[ci];
  FastArgs f = make_fast_args(a, tab32, a16);
  f.items = p.d_items_sorted + C.offset;
  f.n_items = C.n_items;
  const int g = std::max(1, std::min(C.n_items, grid > 0 ? grid : C.grid));
  switch (p.KS) {
    case 2: return launch_class_w<R, 2, MP, WS>(C, f, g, W, p.d_queue + ci, a.stream);
    case 3: return launch_class_w<R, 3, MP, WS>(C, f, g, W, p.d_queue + ci, a.stream);
    case 4: return launch_class_w<R, 4, MP, WS>(C, f, g, W, p.d_queue + ci, a.stream);
    default: break;
  }
  fast_set_error("no persistent kernel instance for this shape");
  return hipErrorNotSupported;
}

}  // namespace
}  // namespace fastk
}  // namespace sf
