// Equality-only QP layer of the decoders (Sec. IV: the QP of eq. sf_form without its inequality
// rows, which has a closed form) and its reverse mode.
//
// xi_out = argmin 1/2 ||xi - xi_in||^2 subject to the boundary rows A xi = b of eq. boundary_con.
// Those rows touch only the three first and three last coefficients of each robot-axis (the
// Bernstein end conditions), and restricted to them A is the invertible 6 x 6 block whose inverse
// sf_setup stores as Bmap.  So the free coefficients pass through and the six pinned ones become
// Bmap b.  The kernels stream the coefficients (HBM-bound), each thread owning fixed positions of the samples
// of a chunk.
#include "sf_eqqp.h"

#include <algorithm>
#include <mutex>

namespace sf {
namespace {

constexpr int kEqBlock = 512;

// 16-byte accesses where the sample's size and the pointers allow, else single elements.
template <typename T, int VW> struct Vec { typedef T type __attribute__((ext_vector_type(VW))); };

// The positions (groups of VW elements of a sample) of this thread and the samples it visits: a position is
// a thread's for the whole chunk, so its role and pinned values (or sums) stay in registers.  With at most
// kEqBlock positions the workgroup covers `step` samples at a time, else it walks the positions.
template <typename F>
__device__ __forceinline__ void for_positions(int nV, F body) {
  if (nV <= kEqBlock) {
    const int step = kEqBlock / nV, s0 = threadIdx.x / nV;
    if (s0 < step) body(threadIdx.x - s0 * nV, s0, step);
  } else {
    for (int ev = threadIdx.x; ev < nV; ev += kEqBlock) body(ev, 0, 1);
  }
}

// Pinned slot of position e of a sample (row * 6 + r), -1: a free coefficient.
__device__ __forceinline__ int eq_slot(int e, int m) {
  const int row = e / m, k = e - row * m;
  const int r = k < 3 ? k : (k >= m - 3 ? k - (m - kNFix) : -1);
  return r < 0 ? -1 : row * kNFix + r;
}

// One chunk of the forward: free coefficients pass, pinned ones become Bmap b.  Four accesses in flight per
// thread.  16 robots x 2^19 samples: 0.43 ms, 5.1 TB/s, the rate of a device copy.
template <typename T, int VW>
__device__ void eq_forward(int nDm, int m, int count, const T* __restrict__ Bmap, const T* __restrict__ bv, const T* xin,
                           T* xout) {
  typedef typename Vec<T, VW>::type V;
  const int nV = nDm / VW;
  for_positions(nV, [&](int ev, int s0, int step) {
    T pin[VW];
    bool fix[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      const int slot = eq_slot(ev * VW + j, m);
      fix[j] = slot >= 0;
      T acc = T(0);
      if (fix[j]) {
        const int row = slot / kNFix, r = slot - row * kNFix;
        for (int s = 0; s < kNFix; ++s) acc = fma(Bmap[r * kNFix + s], bv[row * kNFix + s], acc);
      }
      pin[j] = acc;
    }
    const V* in = reinterpret_cast<const V*>(xin) + ev;
    V* out = reinterpret_cast<V*>(xout) + ev;
    auto put = [&](int s, V v) {
#pragma unroll
      for (int j = 0; j < VW; ++j) v[j] = fix[j] ? pin[j] : v[j];
      out[(int64_t)s * nV] = v;
    };
    int s = s0;
    for (; s + 3 * step < count; s += 4 * step) {
      V v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = in[(int64_t)(s + u * step) * nV];
#pragma unroll
      for (int u = 0; u < 4; ++u) put(s + u * step, v[u]);
    }
    for (; s < count; s += step) put(s, in[(int64_t)s * nV]);
  });
}

// One chunk of the reverse mode in one pass: g_xi_in = g with the pinned positions zeroed (g_in may be NULL
// or g itself), and per pinned slot the sum of g over the chunk's samples (part may be NULL), in a fixed
// order: a thread's samples, then the `step` threads of a position in order (red: kEqBlock VW elements).
// The sums and the zeroed copy in two kernels read g twice: 16 robots x 2^19 samples 0.65 ms, now 0.43 ms.
template <typename T, int VW>
__device__ void eq_reverse(int nDm, int m, int count, const T* g, T* g_in, T* __restrict__ part, T* red) {
  typedef typename Vec<T, VW>::type V;
  const int nV = nDm / VW;
  for_positions(nV, [&](int ev, int s0, int step) {
    bool fix[VW];
    T sum[VW];
#pragma unroll
    for (int j = 0; j < VW; ++j) {
      fix[j] = eq_slot(ev * VW + j, m) >= 0;
      sum[j] = T(0);
    }
    const V* in = reinterpret_cast<const V*>(g) + ev;
    V* out = reinterpret_cast<V*>(g_in) + ev;
    auto put = [&](int s, V v) {
#pragma unroll
      for (int j = 0; j < VW; ++j) {
        sum[j] += v[j];
        v[j] = fix[j] ? T(0) : v[j];
      }
      if (g_in) out[(int64_t)s * nV] = v;
    };
    int s = s0;
    for (; s + 3 * step < count; s += 4 * step) {
      V v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = in[(int64_t)(s + u * step) * nV];
#pragma unroll
      for (int u = 0; u < 4; ++u) put(s + u * step, v[u]);
    }
    for (; s < count; s += step) put(s, in[(int64_t)s * nV]);
    if (part) {
#pragma unroll
      for (int j = 0; j < VW; ++j) {
        if (step > 1) red[threadIdx.x * VW + j] = sum[j];
        else if (fix[j]) part[eq_slot(ev * VW + j, m)] = sum[j];
      }
    }
  });
  if (part && nV <= kEqBlock && kEqBlock / nV > 1) {
    __syncthreads();
    const int step = kEqBlock / nV;
    for (int e = threadIdx.x; e < nDm; e += kEqBlock) {
      const int slot = eq_slot(e, m);
      if (slot < 0) continue;
      T acc = red[e];
      for (int q = 1; q < step; ++q) acc += red[q * nDm + e];
      part[slot] = acc;
    }
    __syncthreads();
  }
}

// Forward: one workgroup per chunk of samples of one problem (grid-stride over the chunks).
template <typename T>
__global__ void __launch_bounds__(kEqBlock)
qp_equality_kernel(const DevCfg* __restrict__ cfgs, const T* __restrict__ tab, const DevProblem* __restrict__ probs,
                   const WorkItem* __restrict__ chunks, int n_chunks, const T* xin, const T* __restrict__ bvals,
                   T* xout) {
  constexpr int VW = 16 / sizeof(T);
  for (int it = blockIdx.x; it < n_chunks; it += gridDim.x) {
    const WorkItem w = chunks[it];
    const DevProblem pr = probs[w.problem];
    const DevCfg& c = cfgs[pr.cfg];
    const int m = c.m, nDm = c.n * c.D * m;
    const T* in = xin + pr.coef_off + (int64_t)w.first * nDm;
    T* out = xout + pr.coef_off + (int64_t)w.first * nDm;
    const bool vec = nDm % VW == 0 && (uintptr_t)in % 16 == 0 && (uintptr_t)out % 16 == 0;
    if (vec) eq_forward<T, VW>(nDm, m, w.count, tab + c.off_Bmap, bvals + pr.bnd_off, in, out);
    else eq_forward<T, 1>(nDm, m, w.count, tab + c.off_Bmap, bvals + pr.bnd_off, in, out);
  }
}

// Reverse mode, part 1: the zeroed copy and the chunks' sums.  g_bvals is linear in these sums.
template <typename T>
__global__ void __launch_bounds__(kEqBlock)
qp_equality_bwd_kernel(const DevCfg* __restrict__ cfgs, const DevProblem* __restrict__ probs,
                       const WorkItem* __restrict__ chunks, int n_chunks, const T* g, T* g_in, T* __restrict__ part,
                       int part_stride) {
  constexpr int VW = 16 / sizeof(T);
  __shared__ T red[kEqBlock * VW];
  for (int it = blockIdx.x; it < n_chunks; it += gridDim.x) {
    const WorkItem w = chunks[it];
    const DevProblem pr = probs[w.problem];
    const DevCfg& c = cfgs[pr.cfg];
    const int m = c.m, nDm = c.n * c.D * m;
    const T* in = g + pr.coef_off + (int64_t)w.first * nDm;
    T* out = g_in ? g_in + pr.coef_off + (int64_t)w.first * nDm : nullptr;
    T* sums = part ? part + (int64_t)it * part_stride : nullptr;
    const bool vec = nDm % VW == 0 && (uintptr_t)in % 16 == 0 && (uintptr_t)out % 16 == 0;
    if (vec) eq_reverse<T, VW>(nDm, m, w.count, in, out, sums, red);
    else eq_reverse<T, 1>(nDm, m, w.count, in, out, sums, red);
  }
}

// Reverse mode, part 2: one workgroup per (problem, robot-axis row) sums the row's six slots over the problem's
// chunks and writes g_bvals[row][col] = sum_r Bmap[r][col] G[r].  A lane owns (chunk of ten, slot), so that a
// row's slots, contiguous in a chunk's sums, are read together, once; fixed order.  Bound by the latency of
// the strided reads: 8457 chunks of 16 robots took 70 us with a wave per slot, 27 us now.
constexpr int kSumWaves = 16, kSumChunks = 10;   // per workgroup, per wave
template <typename T>
__global__ void __launch_bounds__(64 * kSumWaves)
qp_equality_bsum_kernel(const DevCfg* __restrict__ cfgs, const T* __restrict__ tab,
                        const DevProblem* __restrict__ probs, int n_probs, const int* __restrict__ chunk_first,
                        const T* __restrict__ part, int part_stride, T* __restrict__ g_bvals) {
  __shared__ T red[kSumWaves][kSumChunks * kNFix];
  __shared__ T G[kNFix];
  const int row = blockIdx.x;
  for (int p = blockIdx.y; p < n_probs; p += gridDim.y) {
    const DevProblem pr = probs[p];
    const DevCfg& c = cfgs[pr.cfg];
    if (row >= c.n * c.D) continue;               // uniform over the workgroup
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane < kSumChunks * kNFix) {
      constexpr int kStep = kSumWaves * kSumChunks;
      const T* src = part + row * kNFix + lane % kNFix;
      const int end = chunk_first[p + 1];
      T a[4] = {T(0), T(0), T(0), T(0)};
      int ch = chunk_first[p] + wave * kSumChunks + lane / kNFix;
      for (; ch + 3 * kStep < end; ch += 4 * kStep) {
        T v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = src[(int64_t)(ch + kStep * u) * part_stride];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] += v[u];
      }
      for (; ch < end; ch += kStep) a[0] += src[(int64_t)ch * part_stride];
      red[wave][lane] = (a[0] + a[1]) + (a[2] + a[3]);
    }
    __syncthreads();
    if (wave == 0) {
      T v = T(0);
      if (lane < kSumChunks * kNFix)
        for (int ww = 0; ww < kSumWaves; ++ww) v += red[ww][lane];
      T acc = v;
      for (int q = 1; q < kSumChunks; ++q) acc += __shfl(v, lane + q * kNFix);
      if (lane < kNFix) G[lane] = acc;
    }
    __syncthreads();
    if (threadIdx.x < kNFix) {
      const T* Bmap = tab + c.off_Bmap;
      T v = T(0);
      for (int q = 0; q < kNFix; ++q) v = fma(Bmap[q * kNFix + threadIdx.x], G[q], v);
      g_bvals[pr.bnd_off + row * kNFix + threadIdx.x] = v;
    }
    __syncthreads();
  }
}

// Allocation-free reverse mode: the tables of a batch, built on the device from its (config slot,
// sample count) list, in the layout and order of the host-built plan (get_plan / get_eq_chunks):
// problems packed in order, chunks of eq_chunk_samples samples.
__global__ void __launch_bounds__(256)
eq_noalloc_tables_kernel(const DevCfg* __restrict__ cfgs, EqNoAllocBatch b, DevProblem* __restrict__ probs,
                         WorkItem* __restrict__ chunks, int32_t* __restrict__ chunk_first) {
  __shared__ int32_t first[kEqNoAllocMaxProblems + 1], per[kEqNoAllocMaxProblems];
  if (threadIdx.x == 0) {
    int64_t coef = 0, bnd = 0, smp = 0;
    int32_t ch = 0;
    for (int p = 0; p < b.n_probs; ++p) {
      const DevCfg& c = cfgs[b.slot[p]];
      DevProblem pr;
      pr.cfg = b.slot[p];
      pr.count = b.count[p];
      pr.coef_off = coef;
      pr.bnd_off = bnd;
      pr.sample_base = smp;
      probs[p] = pr;
      per[p] = eq_chunk_samples(b.count[p], c.n * c.D * c.m, b.want);
      first[p] = ch;
      chunk_first[p] = ch;
      ch += (b.count[p] + per[p] - 1) / per[p];
      coef += (int64_t)b.count[p] * c.n * c.D * c.m;
      bnd += (int64_t)c.n * c.D * kNFix;
      smp += b.count[p];
    }
    first[b.n_probs] = ch;
    chunk_first[b.n_probs] = ch;
  }
  __syncthreads();
  for (int p = 0; p < b.n_probs; ++p)
    for (int q = threadIdx.x; q < first[p + 1] - first[p]; q += blockDim.x) {
      const int s = q * per[p];
      chunks[first[p] + q] = WorkItem{p, s, min(per[p], b.count[p] - s), 0};
    }
}

// The array itself.  Host code never uses its name as an address: hipGetSymbolAddress gives each
// device's copy, kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[kEqNoAllocBytes];

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mu;

}  // namespace

EqNoAllocLayout eq_noalloc_layout(int32_t n_probs, int32_t n_chunks, int32_t part_stride, size_t elem) {
  auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
  EqNoAllocLayout l;
  l.probs = 0;
  l.chunks = up(l.probs + (size_t)n_probs * sizeof(DevProblem));
  l.chunk_first = up(l.chunks + (size_t)n_chunks * sizeof(WorkItem));
  l.part = up(l.chunk_first + (size_t)(n_probs + 1) * sizeof(int32_t));
  l.total = l.part + (size_t)n_chunks * part_stride * elem;
  return l;
}

hipError_t eq_noalloc_init(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[device]) return hipSuccess;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = p;
  return hipSuccess;
}

void* eq_noalloc_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return g_scratch_ptr[device];
}

hipError_t launch_eq_noalloc_tables(const DevCfg* cfgs, const EqNoAllocBatch& b, void* base,
                                    const EqNoAllocLayout& lay, hipStream_t stream) {
  unsigned char* s = static_cast<unsigned char*>(base);
  hipLaunchKernelGGL(eq_noalloc_tables_kernel, dim3(1), dim3(256), 0, stream, cfgs, b,
                     reinterpret_cast<DevProblem*>(s + lay.probs), reinterpret_cast<WorkItem*>(s + lay.chunks),
                     reinterpret_cast<int32_t*>(s + lay.chunk_first));
  return hipGetLastError();
}

template <typename T>
hipError_t launch_qp_equality(const EqArgs& a) {
  if (a.n_chunks == 0) return hipSuccess;
  const int grid = a.n_chunks;
  if (a.forward) {
    hipLaunchKernelGGL(qp_equality_kernel<T>, dim3(grid), dim3(kEqBlock), 0, a.stream, a.cfgs,
                       static_cast<const T*>(a.tab), a.probs, a.chunks, a.n_chunks, static_cast<const T*>(a.in),
                       static_cast<const T*>(a.bvals), static_cast<T*>(a.out));
    return hipGetLastError();
  }
  T* part = a.g_bvals ? static_cast<T*>(a.part) : nullptr;
  hipLaunchKernelGGL(qp_equality_bwd_kernel<T>, dim3(grid), dim3(kEqBlock), 0, a.stream, a.cfgs, a.probs, a.chunks,
                     a.n_chunks, static_cast<const T*>(a.in), static_cast<T*>(a.out), part, a.part_stride);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !part) return e;
  hipLaunchKernelGGL(qp_equality_bsum_kernel<T>, dim3(a.max_rows, std::min(a.n_probs, 65535)),
                     dim3(64 * kSumWaves), 0,
                     a.stream, a.cfgs, static_cast<const T*>(a.tab), a.probs, a.n_probs, a.chunk_first, part,
                     a.part_stride, static_cast<T*>(a.g_bvals));
  return hipGetLastError();
}

template hipError_t launch_qp_equality<double>(const EqArgs&);
template hipError_t launch_qp_equality<float>(const EqArgs&);

}  // namespace sf
