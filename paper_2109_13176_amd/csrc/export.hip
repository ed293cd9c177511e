// Export kernels: the per-column reductions and the 2D maps of Sec. III-D of
// arXiv 2109.13176, the Sec. III-A lookup table / data array, and its import.
#include <math.h>

#include "export_body.h"

namespace gvom {

namespace {

__global__ __launch_bounds__(kBlock) void k_column(ColumnArgs a) { column_body(a, blockIdx.x); }

// Block b of a surface pass sums super group b of the table export's ranks in
// its last wave (a pass has at least one tile per 64 x 64 columns).
__device__ __forceinline__ void surface_rank_sums(const SurfaceArgs& a, const int b) {
  if (64 * b < a.rank_n && threadIdx.x >= kSurfThreads - 64)
    super_sum_body(a.rank_cnt, a.rank_n, a.rank_sum, b);
}

template <int TILE>
__global__ __launch_bounds__(kSurfThreads, 8) void k_surface(SurfaceArgs a, int H) {
  const bool wild = *a.imported & kWild;  // (before any store: a scalar load)
  surface_rank_sums(a, blockIdx.x * gridDim.y + blockIdx.y);
  surface_body<kSurfThreads, TILE>(a, wild, H, blockIdx.x, blockIdx.y);
}

__global__ __launch_bounds__(kBlock) void k_lut_count(LutArgs a) { lut_count_body(a, blockIdx.x); }

__global__ __launch_bounds__(kBlock) void k_lut_sums(int32_t* cnt, int n, int32_t* sum) {
  const int g = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  if (64 * g < n) super_sum_body(cnt, n, sum, g);
}

__global__ __launch_bounds__(1024) void k_lut_scan(int32_t* base, int nb, int64_t* n_occupied) {
  lut_scan_body<1024>(base, nb, n_occupied);
}

__global__ __launch_bounds__(kBlock) void k_lut_write(LutArgs a, uint32_t nz_magic) {
  lut_write_body(a, nz_magic, blockIdx.x, blockIdx.y);  // brick row, group of 4 bricks
}

// Density of every voxel (the voxel-map output, Fig. 1), in window-local
// table order, one region per block.  The hits are read for the occupied
// voxels only, whose densities take the place of their passes in LDS.
//
// Bound: HBM, 4 V read (passes) + 4 V written.  Measured at 512 x 512 x 64:
// 31.4 us (201 MB, the hits of every voxel read) -> 24.5 us (134 MB).
__global__ __launch_bounds__(kBlock) void k_density(DensityArgs a, uint32_t nz_magic) {
  extern __shared__ __attribute__((aligned(16))) int32_t lpass[];  // [64][lut_row(nz)]
  __shared__ RegionCols rc;
  const int nz = a.d.nz, nzp = lut_row(nz);
  region_load(a.d, a.passes, a.occ, nz_magic, blockIdx.x, blockIdx.y, lpass, rc,
              [](int, int32_t) {});
  __syncthreads();
  const int nocc = rc.pre[kRegCols];
  for (int o = threadIdx.x; o < nocc; o += kBlock) {
    int r, z;
    const int t = region_voxel(rc, o, r, z);
    const double h = a.hits[rc.base[t] + ((int64_t)wrap_add(z + a.d.ro[2], nz) << 4)];
    const double p = lpass[t * nzp + z];
    lpass[t * nzp + z] = __float_as_int((float)(h / (h + p)));
  }
  __syncthreads();
  const bool vec = (nz & 3) == 0 && ((uintptr_t)a.out & 15) == 0;
  region_quads(rc, nz, [&](int t, int q) {
    const Mask128 mt = {rc.lo[t], rc.hi[t]};
    const int z0 = 4 * q;
    const int4 pv = *(const int4*)(lpass + t * nzp + z0);
    const int32_t p4[4] = {pv.x, pv.y, pv.z, pv.w};
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const bool occ = z0 + e < nz && test_bit(mt, z0 + e);
      v[e] = occ ? __int_as_float(p4[e]) : p4[e] >= 1 ? 0.0f : __uint_as_float(kQNaN);
    }
    store_quad(a.out + (int64_t)rc.col[t] * nz + z0, v, nz - z0, vec);
  });
}

// Per-column features (FeatArgs), one region per block: the passes summed from
// the LDS rows (four threads per column), the occupied voxels' hits and lowest
// returns added one thread per voxel (integer sums: any order), then four
// features per thread.
//
// Bound: HBM, 4 V read + 64 C written.  Measured at 512 x 512 x 64: 87 us (one
// lane per column, hits and passes of every voxel in 4-byte reads 16 bytes
// apart) -> 22.8 us.  With few levels the round trips of a region bound it, so the 2D
// maps are loaded beside the region's words: 2048 x 2048 x 8 227 us (a lane per column),
// 189 (2D maps last), 155; 4096 x 4096 x 4 596, 688, 624; 4096 x 4096 x 1 376, 680, 596.
__global__ __launch_bounds__(kBlock) void k_features(FeatArgs a, uint32_t nz_magic) {
  extern __shared__ __attribute__((aligned(16))) int32_t lpass[];  // [64][lut_row(nz)]
  __shared__ RegionCols rc;
  __shared__ unsigned long long sh[kRegCols], sq[kRegCols];  // sums of hits, of lowest returns
  __shared__ int32_t top_q[kRegCols], bot_h[kRegCols], bot_p[kRegCols];
  static_assert(kBlock == 4 * kRegCols, "four threads per column");
  const int ny = a.d.ny, nz = a.d.nz, nzp = lut_row(nz);
  const int t = threadIdx.x >> 2, part = threadIdx.x & 3;
  // the 2D maps of the thread's column, beside the region's loads
  int32_t sxc, syc;
  const int32_t c0 = max(region_col(a.d, blockIdx.x, blockIdx.y, t, sxc, syc), 0);
  const float m0 = (part == 2 ? a.density : a.height)[c0], m1 = a.slope[c0], m2 = a.rough[c0];
  const uint8_t fl0 = a.flags[c0];
  const bool thin0 = a.thin && a.thin[c0];
  region_load(a.d, a.passes, a.occ, nz_magic, blockIdx.x, blockIdx.y, lpass, rc,
              [&](int t, int32_t) { sh[t] = sq[t] = 0ull; });
  __syncthreads();
  const int nocc = rc.pre[kRegCols];
  for (int o = threadIdx.x; o < nocc; o += kBlock) {
    int r, z;
    const int t = region_voxel(rc, o, r, z);
    const int64_t e = rc.base[t] + ((int64_t)wrap_add(z + a.d.ro[2], nz) << 4);
    const int32_t h = a.hits[e], q = a.minqz[e];
    atomicAdd(&sh[t], (unsigned long long)(int64_t)h);
    atomicAdd(&sq[t], (unsigned long long)(int64_t)q);
    if (r == 0) {
      bot_h[t] = h;
      bot_p[t] = lpass[t * nzp + z];
    }
    if (o + 1 == rc.pre[t + 1]) top_q[t] = q;
  }
  int64_t sp = 0;
  for (int q = part; 4 * q < nz; q += 4) {
    const int4 v = *(const int4*)(lpass + t * nzp + 4 * q);
    sp += v.x;
    if (4 * q + 1 < nz) sp += v.y;
    if (4 * q + 2 < nz) sp += v.z;
    if (4 * q + 3 < nz) sp += v.w;
  }
  sp += __shfl_xor(sp, 1);
  sp += __shfl_xor(sp, 2);
  __syncthreads();
  const int32_t c = rc.col[t];
  if (c < 0) return;
  const int x = c / ny, y = c - x * ny;
  const int cnt = rc.pre[t + 1] - rc.pre[t];
  const bool thinned = thin0;
  const double q2m = a.res / 65536.0;
  float f[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  const uint8_t fl = thinned ? 0 : fl0;
  if (part == 0) {
    if (!thinned) {
      f[0] = (float)(double)(int64_t)sh[t];
      f[1] = (float)(double)sp;
      f[2] = (float)cnt;
      f[3] = (float)((double)cnt / (double)nz);
    }
  } else if (part == 1) {
    if (fl & 1) {
      f[0] = m0;
      f[3] = 1.0f;
    }
    if (!thinned && cnt > 0) {
      f[1] = (float)((double)top_q[t] * q2m);
      f[2] = (float)(((double)(int64_t)sq[t] / (double)cnt) * q2m);
    }
  } else if (part == 2) {
    if (!thinned && cnt > 0) {
      const double hb = bot_h[t], pb = bot_p[t];
      f[0] = (float)(hb / (hb + pb));
    }
    if (fl & 2) f[1] = m0;
    if (fl & 32) {
      f[2] = m1;
      f[3] = m2;
    }
  } else {
    if (fl & 32) f[0] = 1.0f;
    const double cx = ((double)(a.O[0] + x) + 0.5) * a.res - a.sx;
    const double cy = ((double)(a.O[1] + y) + 0.5) * a.res - a.sy;
    f[1] = (float)sqrt(cx * cx + cy * cy);
    if (fl & 1) f[2] = (float)(a.sz - (double)m0);
    if (thinned) f[3] = 1.0f;
  }
  float* o = a.feat + (int64_t)c * 16 + 4 * part;
  if (((uintptr_t)a.feat & 15) == 0) {
    *(float4*)o = make_float4(f[0], f[1], f[2], f[3]);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++) o[e] = f[e];
  }
}

// Empties the columns marked in `thin` (window-local; null: every column),
// one storage region per block: the passes words that hold a count are
// zeroed, hits and lowest returns only where the occupancy words have a
// voxel (they are empty elsewhere), then the columns' words.
//
// Bound: HBM, 4 V read.  Measured at 512 x 512 x 64: half the columns 141 us
// (4-byte stores to every voxel) -> 14.5 us; the whole map 3 x 18.3 us (three
// fills) -> 14.5 us.
//
// NT: threads per block.  A region of nz levels has 16 nz words, so one wave takes those
// of few levels (with four, most do nothing but be launched).  The whole map by calls,
// 256 / 64 threads: 4096 x 4096 x 4 250 / 104 us, 2048 x 2048 x 16 95 / 62, 512 x 512 x 32
// 22.9 / 23.4, 512 x 512 x 64 28.4 / 32.1.
template <int NT>
__global__ __launch_bounds__(NT) void k_thin(Dims d, const uint8_t* thin, int32_t* hits,
                                                 int32_t* passes, int32_t* minqz,
                                                 unsigned long long* occ, uint32_t nz_magic) {
  __shared__ unsigned long long lo[kRegCols], hi[kRegCols];  // storage z order, marked columns
  __shared__ unsigned long long marked;
  const int nz = d.nz, tid = threadIdx.x, bxr = blockIdx.x, byr = blockIdx.y;
  const int64_t r0 = col_base(d, 4 * bxr, 16 * byr);
  const int nv4 = min(4, d.nby - 4 * byr) * nz * 4;
  if (tid < kRegCols) {
    int sx, sy;
    const int32_t c = region_col(d, bxr, byr, tid, sx, sy);
    const bool on = c >= 0 && (!thin || thin[c]);
    unsigned long long w0 = 0ull, w1 = 0ull;
    if (on) {
      const int64_t col = ((int64_t)sx * d.ny + sy) * d.W;
      w0 = occ[col];
      if (d.W > 1) w1 = occ[col + 1];
      if (w0) occ[col] = 0ull;
      if (w1) occ[col + 1] = 0ull;
    }
    lo[tid] = w0;
    hi[tid] = w1;
    const unsigned long long b = __ballot(on);
    if (tid == 0) marked = b;
  }
  __syncthreads();
  const unsigned long long mk = marked;
  if (!mk) return;
  for (int k0 = 0; k0 < nv4; k0 += kLutLoads * NT) {
    int4 v[kLutLoads];
#pragma unroll
    for (int u = 0; u < kLutLoads; u++)
      v[u] = ((const int4*)(passes + r0))[min(k0 + u * NT + tid, nv4 - 1)];
#pragma unroll
    for (int u = 0; u < kLutLoads; u++) {
      const int k4 = k0 + u * NT + tid;
      if (k4 >= nv4) continue;
      int zs;
      const int t = region_word(k4, nz, nz_magic, zs);
      const unsigned long long m = mk >> t;  // bits 0, 16, 32, 48: the word's columns
      const bool on[4] = {(m & 1ull) != 0, ((m >> 16) & 1ull) != 0, ((m >> 32) & 1ull) != 0,
                          ((m >> 48) & 1ull) != 0};
      const int32_t p[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
      const int32_t n[4] = {on[0] ? 0 : p[0], on[1] ? 0 : p[1], on[2] ? 0 : p[2], on[3] ? 0 : p[3]};
      const int64_t s = r0 + 4 * (int64_t)k4;
      if ((p[0] ^ n[0]) | (p[1] ^ n[1]) | (p[2] ^ n[2]) | (p[3] ^ n[3]))
        *(int4*)(passes + s) = make_int4(n[0], n[1], n[2], n[3]);
      const unsigned long long* w = zs < 64 ? lo : hi;
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if ((w[t + 16 * e] >> (zs & 63)) & 1ull) {
          hits[s + e] = 0;
          minqz[s + e] = INT32_MAX;
        }
      }
    }
  }
}

// Costmap: one lane per pixel, the weighted layers added in a fixed order
// in binary32.
__global__ __launch_bounds__(kBlock) void k_costmap(CostArgs a) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= a.n) return;
  const float sl = a.slope[i], ro = a.rough[i], de = a.density[i];
  const uint32_t f = a.flags[i];
  float c = 0.0f;
  if (!isnan(sl)) c = c + a.w[0] * sl;
  if (!isnan(ro)) c = c + a.w[1] * ro;
  if (!isnan(de)) c = c + a.w[2] * de;
  if (f & 2u) c = c + a.w[3];
  if (f & 4u) c = c + a.w[4];
  if (f & 8u) c = c + a.w[5];
  if (f & 16u) c = c + a.w[6];
  if (!(f & 1u)) c = c + a.w[7];
  a.cost[i] = c;
}

// Import, one region per block: the table's columns are read in 16-byte words
// into the LDS rows, then the region is written in storage order, the records
// of occupied voxels gathered on the way.  Hits and lowest returns are written
// where the old or the new map has an occupied voxel (they are empty
// elsewhere).  err receives kBadContent (the caller then empties the map) and
// kWild.
//
// Bound: HBM, 4 V read + 4 V written.  Measured at 512 x 512 x 64: 237 us (a
// lane per voxel of a column, each storing to lines of its own) -> 38.7 us.
__global__ __launch_bounds__(kBlock) void k_import(Dims d, const int32_t* __restrict__ lut,
                                                   const map_voxel_t* __restrict__ data,
                                                   int64_t n_data, int32_t* hits, int32_t* passes,
                                                   int32_t* minqz, unsigned long long* occ,
                                                   int32_t origin_z, int32_t* err,
                                                   uint32_t nz_magic) {
  extern __shared__ __attribute__((aligned(16))) int32_t lval[];  // [64][lut_row(nz)]
  __shared__ unsigned long long oldw[2][kRegCols], neww[2][kRegCols];  // storage z order
  __shared__ int32_t scol[kRegCols];
  __shared__ int32_t found;
  const int nz = d.nz, roz = d.ro[2], nzp = lut_row(nz);
  const int tid = threadIdx.x, bxr = blockIdx.x, byr = blockIdx.y;
  int64_t wcol = -1;
  if (tid == 0) found = 0;
  if (tid < kRegCols) {
    int sx, sy;
    const int32_t c = region_col(d, bxr, byr, tid, sx, sy);
    scol[tid] = c;
    wcol = c >= 0 ? ((int64_t)sx * d.ny + sy) * d.W : -1;
    oldw[0][tid] = wcol >= 0 ? occ[wcol] : 0ull;
    oldw[1][tid] = wcol >= 0 && d.W > 1 ? occ[wcol + 1] : 0ull;
    neww[0][tid] = neww[1][tid] = 0ull;
  }
  __syncthreads();
  // table words (column slot t, quad q), as region_quads; columns outside the
  // map read as empty voxels
  const int nq = (nz + 3) >> 2;
  const int qsh = nq > 1 ? 32 - __clz(nq - 1) : 0;
  const bool vec = (nz & 3) == 0 && ((uintptr_t)lut & 15) == 0;
  for (int i0 = 0; i0 < (kRegCols << qsh); i0 += kLutLoads * kBlock) {
    int4 v[kLutLoads];
#pragma unroll
    for (int u = 0; u < kLutLoads; u++) {
      const int i = i0 + u * kBlock + tid;
      const int t = (i >> qsh) & (kRegCols - 1), q = min(i & ((1 << qsh) - 1), nq - 1);
      const int32_t* src = lut + (int64_t)max(scol[t], 0) * nz + 4 * q;
      if (vec) {
        v[u] = *(const int4*)src;
      } else {
        const int last = nz - 1 - 4 * q;  // clamped: every lane loads in bounds
        v[u] = make_int4(src[0], src[min(1, last)], src[min(2, last)], src[min(3, last)]);
      }
    }
#pragma unroll
    for (int u = 0; u < kLutLoads; u++) {
      const int i = i0 + u * kBlock + tid;
      const int t = i >> qsh, q = i & ((1 << qsh) - 1);
      if (t < kRegCols && q < nq)
        *(int4*)(lval + t * nzp + 4 * q) = scol[t] >= 0 ? v[u] : make_int4(-1, -1, -1, -1);
    }
  }
  __syncthreads();
  const int64_t r0 = col_base(d, 4 * bxr, 16 * byr);
  const int nv4 = min(4, d.nby - 4 * byr) * nz * 4;
  int32_t f = 0;
  for (int k4 = tid; k4 < nv4; k4 += kBlock) {
    int zs;
    const int t = region_word(k4, nz, nz_magic, zs);
    const int lz = zs >= roz ? zs - roz : zs - roz + nz;
    const int32_t* row = lval + t * nzp + lz;
    int32_t h[4] = {0, 0, 0, 0}, p[4], mq[4] = {INT32_MAX, INT32_MAX, INT32_MAX, INT32_MAX};
    bool write = false;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int32_t v = row[16 * e * nzp];
      p[e] = 0;
      write |= (oldw[zs >> 6][t + 16 * e] >> (zs & 63)) & 1ull;
      if (v >= 0) {
        map_voxel_t r = {0, 0, 0};
        if (v < n_data) r = data[v];
        if (r.hits >= 1) {
          h[e] = r.hits;
          p[e] = r.passes;
          mq[e] = r.min_qz;
          write = true;
          atomicOr(&neww[zs >> 6][t + 16 * e], 1ull << (zs & 63));
          if (r.min_qz >> 16 != origin_z + lz) f |= kWild;
        } else {
          f |= kBadContent;
        }
      } else if (v == INT32_MIN) {
        f |= kBadContent;
      } else {
        p[e] = -1 - v;
      }
    }
    const int64_t s = r0 + 4 * (int64_t)k4;
    *(int4*)(passes + s) = make_int4(p[0], p[1], p[2], p[3]);
    if (write) {
      *(int4*)(hits + s) = make_int4(h[0], h[1], h[2], h[3]);
      *(int4*)(minqz + s) = make_int4(mq[0], mq[1], mq[2], mq[3]);
    }
  }
  if (f) atomicOr(&found, f);
  __syncthreads();
  // one update per block, and none once the word has it: with one per voxel, a table
  // given another origin in z (every voxel kWild) took 1.5 ms instead of 0.12
  if (tid == 0 && (found & ~*(volatile const int32_t*)err)) atomicOr(err, found);
  if (wcol >= 0) {
    occ[wcol] = neww[0][tid];
    if (d.W > 1) occ[wcol + 1] = neww[1][tid];
  }
}

// ---- batches: persistent grids over the virtual blocks of all maps
__device__ __forceinline__ int find_map_e(const int32_t* pre, int n, int vb) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (pre[mid] <= vb) lo = mid; else hi = mid;
  }
  return lo;
}

// Completion time of map m: the latest end of its last-stage blocks, kept by
// a fire-and-forget 64-bit max (no fence: only the clock value matters).  A
// persistent block folds consecutive virtual blocks of one map into one
// update, made when it moves on to another map and at its end.
struct Stamper {
  int m = -1;
  unsigned long long end = 0;
  // after the (synchronised) virtual block of map mm; counts only if `last`
  __device__ __forceinline__ void done(int mm, bool last, unsigned long long* stamps) {
    if (threadIdx.x != 0) return;
    if (mm != m) flush(stamps);
    if (last) {
      m = mm;
      end = wall_clock64();
    }
  }
  __device__ __forceinline__ void flush(unsigned long long* stamps) {
    if (threadIdx.x == 0 && m >= 0)
      atomicMax(&stamps[kStampEnds + (blockIdx.x % kStampSlots) * kMaxBatch + m], end);
    m = -1;
  }
};

__global__ __launch_bounds__(kBlock) void k_b_column(const BatchTables* __restrict__ t) {
  const int n = t->st.nmaps;
  const int total = t->st.pre_col[n];
  for (int vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const int m = find_map_e(t->st.pre_col, n, vb);
    column_body(t->col[m], vb - t->st.pre_col[m]);
  }
}

__global__ __launch_bounds__(kSurfThreads, 4) void k_b_surface(const BatchTables* __restrict__ t,
                                                               unsigned long long* stamps) {
  const int n = t->st.nmaps;
  const int total = t->st.pre_surf[n];
  Stamper sp;
  for (int vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const int m = find_map_e(t->st.pre_surf, n, vb);
    const int b = vb - t->st.pre_surf[m];
    const bool wild = *t->sur[m].imported & kWild;
    surface_rank_sums(t->sur[m], b);
    const int ty = t->st.surf_tiles_y[m], H = t->st.surf_H[m], tile = t->st.surf_tile[m];
    if (tile == 64) surface_body<kSurfThreads, 64>(t->sur[m], wild, H, b / ty, b % ty);
    else if (tile == 32) surface_body<kSurfThreads, 32>(t->sur[m], wild, H, b / ty, b % ty);
    else surface_body<kSurfThreads, 16>(t->sur[m], wild, H, b / ty, b % ty);
    __syncthreads();
    sp.done(m, !t->st.last_is_lut[m], stamps);
  }
  sp.flush(stamps);
}

// Scans the sums of the super groups of every map that has many: block b = map b.
// (Every region scanning all of them, a step of two maps of 4096 x 4096 x 4 took 4947 us,
// with this launch 1629.)
__global__ __launch_bounds__(1024) void k_b_lut_scan(const BatchTables* __restrict__ t) {
  const int m = blockIdx.x;
  if (m >= t->st.nmaps || !t->st.last_is_lut[m] || !t->lut[m].scanned) return;
  lut_scan_body<1024>(t->lut[m].super_sum, t->lut[m].nsuper, t->lut[m].n_occupied);
}

__global__ __launch_bounds__(kBlock) void k_b_lut_write(const BatchTables* __restrict__ t,
                                                        unsigned long long* stamps) {
  const int n = t->st.nmaps;
  const int total = t->st.pre_lwrite[n];
  Stamper sp;
  for (int vb = blockIdx.x; vb < total; vb += gridDim.x) {
    const int m = find_map_e(t->st.pre_lwrite, n, vb);
    const int b = vb - t->st.pre_lwrite[m];
    const int by = t->st.lw_by[m];
    lut_write_body(t->lut[m], t->st.nz_magic[m], b / by, b % by);
    __syncthreads();
    sp.done(m, true, stamps);
  }
  sp.flush(stamps);
}

}  // namespace

hipError_t launch_batch_export(const BatchTables* tab, const BatchGrid& g,
                               unsigned long long* stamps, hipStream_t s) {
  if (g.surf_lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_b_surface,
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)g.surf_lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_b_column, dim3(g.col), dim3(kBlock), 0, s, tab);
  hipLaunchKernelGGL(k_b_surface, dim3(g.surf), dim3(kSurfThreads), g.surf_lds, s, tab, stamps);
  if (g.scan) hipLaunchKernelGGL(k_b_lut_scan, dim3(g.scan), dim3(1024), 0, s, tab);
  hipLaunchKernelGGL(k_b_lut_write, dim3(g.lwrite), dim3(kBlock), g.lut_lds, s, tab, stamps);
  return hipGetLastError();
}

hipError_t launch_column(const ColumnArgs& a, hipStream_t s) {
  const int C = a.d.nx * a.d.ny;
  hipLaunchKernelGGL(k_column, dim3((C + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
  return hipGetLastError();
}

size_t surface_lds(int H, int tile) {
  const int T = tile + 2 * H;
  return (size_t)T * surface_stride(T) * 4 + 2 * (size_t)T * surface_mask_stride(T) * 4 +
         2 * (size_t)tile * surface_dist_stride(T) + 2 * (size_t)tile * tile;
}

size_t lut_lds(int nz) { return (size_t)kRegCols * lut_row(nz) * 4; }

// b / nz == umulhi(b, ceil(2^32 / nz)) for every b < 2^20 (here b < 4 * 128)
uint32_t nz_magic(int nz) {
  return nz > 1 ? (uint32_t)((((uint64_t)1 << 32) + (uint64_t)nz - 1) / (uint64_t)nz) : 0u;
}

// A tile's serial phases cost much the same for 16, 32 and 64 pixels, so the
// tile follows the number of compute units: 16 while two blocks per unit hold
// every tile, 64 (which stages 3.2 or, at D = 50, 6.6 cells per pixel where 32
// stages 6.6 or 17) once every unit gets one, else 32.  Measured (us, tiles
// of 16 / 32 / 64, with the events' ~3 us): 128 x 128, D = 13 10.0 / 12.0 / 24.5;
// 354 x 278, D = 20 12.7 / 14.0 / 33; 512 x 512, D = 25 24.3 / 15.8 / 37;
// 640 x 640, D = 50 45 / 35 / 53; 1024 x 1024, D = 50 97 / 72 / 55.
int surface_tile_for(int H, int64_t tiles64, int n_cu) {
  if (8 * tiles64 <= n_cu) return 16;
  return tiles64 >= n_cu && surface_lds(H, 64) <= 160 * 1024 ? 64 : 32;
}

template <int TILE>
hipError_t launch_surface_t(const SurfaceArgs& a, hipStream_t s) {
  const int H = a.search_d > a.half_fit ? a.search_d : a.half_fit;
  const int T = TILE + 2 * H;
  const int MW = (T + 63) / 64;
  if (MW > kMaxMaskWords) return hipErrorInvalidValue;
  const size_t lds = surface_lds(H, TILE);
  if (lds > 160 * 1024) return hipErrorInvalidValue;
  if (lds > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute((const void*)k_surface<TILE>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             (int)lds);
    if (e != hipSuccess) return e;
  }
  dim3 g((a.nx + TILE - 1) / TILE, (a.ny + TILE - 1) / TILE);
  hipLaunchKernelGGL((k_surface<TILE>), g, dim3(kSurfThreads), lds, s, a, H);
  return hipGetLastError();
}

hipError_t launch_surface(const SurfaceArgs& a, int tile, hipStream_t s) {
  return tile == 64 ? launch_surface_t<64>(a, s)
                    : tile == 16 ? launch_surface_t<16>(a, s) : launch_surface_t<32>(a, s);
}

hipError_t launch_lut(const LutArgs& args, bool ranked, hipStream_t s) {
  LutArgs a = args;
  const int C = a.d.nx * a.d.ny;
  const int ng = (C + kGroup - 1) / kGroup;
  const size_t lds = lut_lds(a.d.nz);
  if (!ranked) {
    hipLaunchKernelGGL(k_lut_count, dim3((C + kBlock - 1) / kBlock), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(k_lut_sums, dim3((a.nsuper + 3) / 4), dim3(kBlock), 0, s, a.group_cnt, ng,
                       a.super_sum);
  }
  if (a.nsuper > kWaveSupers) {
    hipLaunchKernelGGL(k_lut_scan, dim3(1), dim3(1024), 0, s, a.super_sum, a.nsuper, a.n_occupied);
    a.scanned = 1;
  }
  dim3 g((a.d.nx + 3) / 4, (a.d.nby + 3) / 4);
  hipLaunchKernelGGL(k_lut_write, g, dim3(kBlock), lds, s, a, nz_magic(a.d.nz));
  return hipGetLastError();
}

dim3 region_grid(const Dims& d) { return dim3((d.nx + 3) / 4, (d.nby + 3) / 4); }

hipError_t launch_density(const DensityArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_density, region_grid(a.d), dim3(kBlock), lut_lds(a.d.nz), s, a,
                     nz_magic(a.d.nz));
  return hipGetLastError();
}

hipError_t launch_features(const FeatArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_features, region_grid(a.d), dim3(kBlock), lut_lds(a.d.nz), s, a,
                     nz_magic(a.d.nz));
  return hipGetLastError();
}

hipError_t launch_thin(const Dims& d, const uint8_t* thin, int32_t* hits, int32_t* passes,
                       int32_t* minqz, unsigned long long* occ, hipStream_t s) {
  if (d.nz <= 16)
    hipLaunchKernelGGL(k_thin<64>, region_grid(d), dim3(64), 0, s, d, thin, hits, passes, minqz,
                       occ, nz_magic(d.nz));
  else
    hipLaunchKernelGGL(k_thin<256>, region_grid(d), dim3(256), 0, s, d, thin, hits, passes, minqz,
                       occ, nz_magic(d.nz));
  return hipGetLastError();
}

hipError_t launch_costmap(const CostArgs& a, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_costmap, dim3((unsigned)((a.n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s,
                     a);
  return hipGetLastError();
}

hipError_t launch_scan_i32(int32_t* base, int nb, int64_t* total, hipStream_t s) {
  hipLaunchKernelGGL(k_lut_scan, dim3(1), dim3(1024), 0, s, base, nb, total);
  return hipGetLastError();
}

hipError_t launch_import(const Dims& d, const int32_t* lut, const map_voxel_t* data,
                         int64_t n_data, int32_t* hits, int32_t* passes, int32_t* minqz,
                         unsigned long long* occ, int32_t origin_z, int32_t* err,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_import, region_grid(d), dim3(kBlock), lut_lds(d.nz), s, d, lut, data, n_data,
                     hits, passes, minqz, occ, origin_z, err, nz_magic(d.nz));
  return hipGetLastError();
}

}  // namespace gvom
