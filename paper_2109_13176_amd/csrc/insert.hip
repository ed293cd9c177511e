// Scan insertion kernels: transform + return binning + exact integer ray
// traversal (Sec. III-C of arXiv 2109.13176), and the slab clears that move
// the toroidal window.
#include <math.h>

#include "insert_body.h"

namespace gvom {

namespace {

// Blocks [0, ray_blocks): the ray pass; the others clear the moved window.
__global__ __launch_bounds__(kRayBlock) void k_rays(InsertArgs a, ClearArgs c, int ray_blocks) {
  const int b = (int)blockIdx.x - ray_blocks;
  if (b < 0) {
    rays_body(a, blockIdx.x);
  } else {
    clear_body(c, (int64_t)b * kRayBlock + threadIdx.x,
               (int64_t)((int)gridDim.x - ray_blocks) * kRayBlock);
  }
}

template <bool DISTINCT>
__global__ __launch_bounds__(kTraceBlock, kTraceWavesPerSimd) void k_trace(InsertArgs a) {
  __shared__ int32_t box_cnt[kBoxCells];
  __shared__ WaveTable wtab[kTraceBlock / 64];
  trace_body<DISTINCT, true, kTraceBlock>(a, blockIdx.x, gridDim.x, box_cnt, wtab);
}

template <bool DISTINCT>
__global__ __launch_bounds__(kBlock) void k_box_fold(InsertArgs a) {
  box_fold_body<DISTINCT>(a, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kRayBlock) void k_clear(ClearArgs a) {
  clear_body(a, (int64_t)blockIdx.x * kRayBlock + threadIdx.x, (int64_t)gridDim.x * kRayBlock);
}

// ---------------------------------------------------------------------------
// Batched stages: persistent grids walk the virtual blocks of all maps of a
// batch; block b of a stage belongs to the map m with pre[m] <= b < pre[m+1].
__device__ __forceinline__ int find_map(const int32_t* pre, int n, int vb) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= vb) lo = mid; else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(kRayBlock) void k_b_rays(const BatchTables* __restrict__ t,
                                                      unsigned long long* stamps) {
  const int n = t->st.nmaps;
  const int total = t->st.pre_rays[n];
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) stamps[0] = wall_clock64();
    // per-map completion maxima, taken by the last stages
    for (int i = kStampEnds + threadIdx.x; i < kStampQueue; i += kRayBlock) stamps[i] = 0;
    if (threadIdx.x == 0) stamps[kStampQueue] = 0;
  }
  for (int vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const int m = find_map(t->st.pre_rays, n, vb);
    const int b = vb - t->st.pre_rays[m], nr = t->st.ray_blocks[m];
    if (b < nr) {
      rays_body(t->ins[m], b);
      __syncthreads();
    } else {
      const int nc = t->st.pre_rays[m + 1] - t->st.pre_rays[m] - nr;
      clear_body(t->clr[m], (int64_t)(b - nr) * kRayBlock + threadIdx.x, (int64_t)nc * kRayBlock);
    }
  }
}

// The blocks' work differs by an order of magnitude (segments per ray, line tables that
// fill up), so each takes its next virtual block from a queue (cleared by the ray pass);
// the answer has the block's time to arrive.  Fixed shares of 1792 virtual blocks per
// map: 922 us for 32 maps, with the queue and fewer of them 648.  (Single items from a
// queue in the single-map kernel, over eight counters: 43 -> 55 us, the counters'
// atomics queue up.)
__global__ __launch_bounds__(kTraceBlock, kTraceWavesPerSimd) void k_b_trace(
    const BatchTables* __restrict__ t, unsigned long long* queue) {
  __shared__ int32_t box_cnt[kBoxCells];
  __shared__ WaveTable wtab[kTraceBlock / 64];
  const int n = t->st.nmaps;
  const int total = t->st.pre_trace[n];
  __shared__ int next;
  for (int vb = blockIdx.x; vb < total; vb = next) {
    // (the answer is needed after the block)
    unsigned long long taken = 0;
    if (threadIdx.x == 0) taken = atomicAdd(queue, 1ull);
    const int m = find_map(t->st.pre_trace, n, vb);
    trace_body<false, true, kTraceBlock>(t->ins[m], vb - t->st.pre_trace[m],
                                         t->ins[m].trace_blocks, box_cnt, wtab);
    if (threadIdx.x == 0) next = (int)(gridDim.x + taken);
    __syncthreads();
  }
}

// Sensor-box folds of every map of the batch: block b = map b / F, fold block
// b mod F (F = kFoldCellBlocks x kFoldGroups).
__global__ __launch_bounds__(kBlock) void k_b_box_fold(const BatchTables* __restrict__ t) {
  constexpr int F = kFoldCellBlocks * kFoldGroups;
  const int m = blockIdx.x / F, f = blockIdx.x - m * F;
  if (m >= t->st.nmaps) return;
  box_fold_body<false>(t->ins[m], f % kFoldCellBlocks, f / kFoldCellBlocks);
}

__global__ __launch_bounds__(kBlock) void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * kBlock)
    p[i] = v;
}

int grid_for(int64_t n) {
  int64_t g = (n + kBlock - 1) / kBlock;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

}  // namespace

int clear_blocks(const ClearArgs& c) {
  if (c.nbox == 0) return 0;
  // two words per thread: the blocks share the device with the ray pass, whose
  // records the next kernel waits for
  const int64_t g = ((int64_t)c.pre[c.nbox] + 2 * kRayBlock - 1) / (2 * kRayBlock);
  return (int)(g < 1 ? 1 : g > 1024 ? 1024 : g);
}

hipError_t launch_clear(const ClearArgs& a, hipStream_t s) {
  if (a.nbox == 0) return hipSuccess;
  // alone on the device: one word, or one column where levels go, per thread (a step
  // of one level on 512 x 512 x 64 13.3 us with the blocks of clear_blocks, 10.0 so)
  int64_t n = a.pre[a.nbox];
  if (a.nslab < a.nbox && n < (int64_t)a.d.nx * a.d.ny) n = (int64_t)a.d.nx * a.d.ny;
  const int64_t g = (n + kRayBlock - 1) / kRayBlock;
  hipLaunchKernelGGL(k_clear, dim3((unsigned)(g < 4096 ? g : 4096)), dim3(kRayBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_batch_insert(const BatchTables* tab, const BatchGrid& g,
                               unsigned long long* stamps, hipStream_t s) {
  hipLaunchKernelGGL(k_b_rays, dim3(g.rays), dim3(kRayBlock), 0, s, tab, stamps);
  hipLaunchKernelGGL(k_b_trace, dim3(g.trace), dim3(kTraceBlock), 0, s, tab,
                     stamps + kStampQueue);
  hipLaunchKernelGGL(k_b_box_fold, dim3(g.fold), dim3(kBlock), 0, s, tab);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, dim3(grid_for(n)), dim3(kBlock), 0, s, p, v, n);
  return hipGetLastError();
}

int64_t max_segments(const Dims& d, int32_t seg_len) {
  int32_t m = d.nx > d.ny ? d.nx : d.ny;
  if (d.nz > m) m = d.nz;
  return (m - 1) / seg_len + 1;
}

hipError_t launch_rays(const InsertArgs& a, const ClearArgs& c, hipStream_t s) {
  if (a.n <= 0) return launch_clear(c, s);
  const int g = (a.n + kRayBlock - 1) / kRayBlock;
  hipLaunchKernelGGL(k_rays, dim3(g + clear_blocks(c)), dim3(kRayBlock), 0, s, a, c, g);
  return hipGetLastError();
}

hipError_t launch_trace(const InsertArgs& a, bool distinct, hipStream_t s) {
  if (a.n <= 0) return hipSuccess;
  if (!a.box_rep || a.trace_blocks < 1) return hipErrorInvalidValue;
  const dim3 fb(kFoldCellBlocks, kFoldGroups);
  if (distinct) {
    hipLaunchKernelGGL(k_trace<true>, dim3(a.trace_blocks), dim3(kTraceBlock), 0, s, a);
    hipLaunchKernelGGL(k_box_fold<true>, dim3(fb), dim3(kBlock), 0, s, a);
  } else {
    hipLaunchKernelGGL(k_trace<false>, dim3(a.trace_blocks), dim3(kTraceBlock), 0, s, a);
    hipLaunchKernelGGL(k_box_fold<false>, dim3(fb), dim3(kBlock), 0, s, a);
  }
  return hipGetLastError();
}

int box_fold_blocks() { return kFoldCellBlocks * kFoldGroups; }

// Sums the ray pass's per-block counters (4 per block) into out[0..3]: one
// block, each thread a strided share of the blocks, then a fixed-order sum
// over the threads (no atomics).
__global__ __launch_bounds__(kBlock) void k_sum_ray_parts(const unsigned long long* parts,
                                                          int64_t nblocks,
                                                          unsigned long long* out) {
  __shared__ unsigned long long s[4][kBlock];
  unsigned long long c[4] = {0, 0, 0, 0};
  for (int64_t b = threadIdx.x; b < nblocks; b += kBlock)
#pragma unroll
    for (int k = 0; k < 4; k++) c[k] += parts[4 * b + k];
#pragma unroll
  for (int k = 0; k < 4; k++) s[k][threadIdx.x] = c[k];
  __syncthreads();
  for (int h = kBlock / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h)
#pragma unroll
      for (int k = 0; k < 4; k++) s[k][threadIdx.x] += s[k][threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x < 4) out[threadIdx.x] = s[threadIdx.x][0];
}

hipError_t launch_sum_ray_parts(const unsigned long long* parts, int64_t nblocks,
                                unsigned long long* out, hipStream_t s) {
  hipLaunchKernelGGL(k_sum_ray_parts, dim3(1), dim3(kBlock), 0, s, parts, nblocks, out);
  return hipGetLastError();
}


}  // namespace gvom
