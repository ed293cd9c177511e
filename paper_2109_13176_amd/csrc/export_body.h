// Device bodies of the export kernels (Sec. III-A and III-D of arXiv
// 2109.13176): the per-column reduction, the slope / roughness /
// negative-obstacle tiles and the lookup-table passes.  Each body does the
// work of one (virtual) block, so the single-map kernels and the batched
// persistent kernel share them.
#pragma once
#include <math.h>

#include "ray_common.h"

namespace gvom {

namespace {

constexpr uint32_t kQNaN = 0x7FC00000u;


// Column occupancy in window-local z order (bit z = local z), nz <= 128.
struct Mask128 {
  unsigned long long lo, hi;
};

__device__ __forceinline__ Mask128 rotate_mask(const unsigned long long w0,
                                               const unsigned long long w1, int nz, int roz) {
  unsigned __int128 m = w0 | (unsigned __int128)w1 << 64;
  if (roz != 0) {
    const unsigned __int128 full =
        nz == 128 ? ~(unsigned __int128)0 : (((unsigned __int128)1 << nz) - 1);
    m = ((m >> roz) | (m << (nz - roz))) & full;
  }
  Mask128 r;
  r.lo = (unsigned long long)m;
  r.hi = (unsigned long long)(m >> 64);
  return r;
}

__device__ __forceinline__ Mask128 local_mask(const unsigned long long* occ, int64_t col,
                                              int W, int nz, int roz) {
  const unsigned long long w0 = occ[col * W], w1 = W > 1 ? occ[col * W + 1] : 0ull;
  return rotate_mask(w0, w1, nz, roz);
}

__device__ __forceinline__ int lowest_bit(const Mask128& m) {
  if (m.lo) return __ffsll((long long)m.lo) - 1;
  if (m.hi) return 64 + __ffsll((long long)m.hi) - 1;
  return -1;
}

__device__ __forceinline__ bool test_bit(const Mask128& m, int z) {
  return z < 64 ? ((m.lo >> z) & 1ull) : ((m.hi >> (z - 64)) & 1ull);
}

// popcount of the bits below z
__device__ __forceinline__ int rank_below(const Mask128& m, int z) {
  if (z < 64) return __popcll(m.lo & ((1ull << z) - 1ull));
  const int zh = z - 64;
  return __popcll(m.lo) + __popcll(m.hi & ((1ull << zh) - 1ull));
}

// Position of the set bit of rank r (0 = lowest) of m; r < popcount(m).
// Halving search: at each width s the bits of the lower s positions are
// counted and the search moves up past them when r is not among them.
__device__ __forceinline__ int select_bit(const Mask128& m, int r) {
  const int pl = __popcll(m.lo);
  unsigned long long w = r < pl ? m.lo : m.hi;
  int pos = r < pl ? 0 : 64;
  r = r < pl ? r : r - pl;
#pragma unroll
  for (int sh = 32; sh >= 1; sh >>= 1) {
    const int c = __popcll(w & ((1ull << sh) - 1ull));
    if (r >= c) {
      r -= c;
      w >>= sh;
      pos += sh;
    }
  }
  return pos;
}

// Inclusive prefix sum over the lanes of a wave (row shifts within 16 lanes,
// then the broadcasts of lanes 15 and 31 of each half).
__device__ __forceinline__ int wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, true);
  return x;
}

// One lane per map column (window-local pixel).  Ground voxel = lowest
// occupied voxel; height = its lowest return.  The positive-obstacle band is
// the occupied voxels n_lo..n_hi above the ground voxel; its density is
// sum(hits) / sum(hits + passes); hard iff that ratio exceeds num/den
// (compared exactly in integers), soft otherwise.
// With a.colpre set it also does the table export's counting pass (the
// occupied voxels of every column, ranked within its group of 64 columns;
// see lut_count_body), from the occupancy mask it loads anyway.
__device__ __forceinline__ void column_counts(const ColumnArgs& a, const int c, const int cnt) {
  const int lane = __lane_id();
  const int incl = wave_scan(cnt);
  const int C = a.d.nx * a.d.ny;
  if (c < C) a.colpre[c] = incl - cnt;
  if (lane == 63 && (c >> 6) * 64 < C) a.group_cnt[c >> 6] = incl;
}

__device__ __forceinline__ void column_body(const ColumnArgs& a, const int blk) {
  const int nx = a.d.nx, ny = a.d.ny, nz = a.d.nz;
  const int c = blk * kBlock + threadIdx.x;
  const bool valid = c < nx * ny;
  int sx = 0, sy = 0;
  Mask128 m = {0ull, 0ull};
  if (valid) {
    const int x = c / ny, y = c - x * ny;
    sx = wrap_add(x + a.d.ro[0], nx);
    sy = wrap_add(y + a.d.ro[1], ny);
    m = local_mask(a.occ, (int64_t)sx * ny + sy, a.d.W, nz, a.d.ro[2]);
  }
  // every lane of the wave takes part in the rank scan
  if (a.colpre) column_counts(a, c, __popcll(m.lo) + __popcll(m.hi));
  const int kg = lowest_bit(m);
  const int64_t base = col_base(a.d, sx, sy);
  int32_t hq = INT32_MIN;
  if (kg >= 0) hq = a.minqz[base + (wrap_add(kg + a.d.ro[2], nz) << 4)];
  float height = __uint_as_float(kQNaN), density = __uint_as_float(kQNaN);
  uint8_t f = 0;
  if (kg >= 0) {
    height = (float)((double)hq * a.res / 65536.0);
    f = 1;
    int64_t sh = 0, sa = 0;
    int cnt = 0;
    const int zlo = kg + a.n_lo;
    const int zhi = min(kg + a.n_hi, nz - 1);
    // the band's occupied levels in chunks of eight, all loads of a chunk in
    // flight before the sums (one memory round trip per chunk)
    for (int z0 = zlo; z0 <= zhi; z0 += 8) {
      int32_t hv[8], pv[8];
#pragma unroll
      for (int u = 0; u < 8; u++) {
        const int z = z0 + u;
        hv[u] = pv[u] = -1;
        if (z <= zhi && test_bit(m, z)) {
          const int64_t e = base + (wrap_add(z + a.d.ro[2], nz) << 4);
          hv[u] = a.hits[e];
          pv[u] = a.passes[e];
        }
      }
#pragma unroll
      for (int u = 0; u < 8; u++) {
        if (hv[u] < 0) continue;
        sh += hv[u];
        sa += (int64_t)hv[u] + pv[u];
        cnt++;
      }
    }
    if (cnt > 0) {
      density = (float)((double)sh / (double)sa);
      const bool hard = sh * a.dens_den > (int64_t)a.dens_num * sa;
      f |= 2 | (hard ? 4 : 8);
    }
  }
  // the defined pixels of the wave's 64 columns, for the surface pass
  const unsigned long long defined = __ballot(hq != INT32_MIN);
  if (!valid) return;
  if ((c & 63) == 0) a.defbits[c >> 6] = defined;
  a.height[c] = height;
  a.density[c] = density;
  a.flags[c] = f;
  a.hq[c] = hq;
}


// 2D surface maps on tiles of TILE x TILE pixels (kPix / NT per thread)
// with a halo of H = max(half_fit, D) pixels staged in LDS.  Defined pixels
// get the N x N least-squares plane (integer normal equations, exact
// determinant, Cramer's rule in double); undefined pixels get the four-cone
// negative-obstacle search.
//
// Cone test: ring d of the +x cone of pixel (x, y) is the slice of staged row
// x+d over columns y-d..y+d; it holds a defined cell iff the distance along
// that row from column y to the nearest defined cell is <= d.  These row
// (and column) distances are precomputed for the tile's own columns (rows)
// from per-line bit masks, so each ring costs one LDS byte; the rings of all
// four cones are looked up together, and so are the defined cells of the four
// stopping slices (about seven in all).
//
// Bound: the latency and VALU issue of a tile's serial phases (there is about
// one tile per compute unit at 512 x 512), not memory (14 bytes per pixel).
// Measured (HIP events): 512 x 512 at 0.2 m 23.5 -> 15.8 us, 1024 x 1024 at
// 0.1 m 108 -> 55 us, 128 x 128 at 0.4 m 15.3 -> 10.0 us, against masks built
// from the staged heights, distances read ring by ring in a layout whose
// column reads met in the same LDS banks, cones and their cells one after the
// other, and 64-bit normal sums in every cell.
constexpr int kSurfThreads = 1024;
constexpr int kMaxMaskWords = 3;  // staged edge <= 192 cells

// LDS row stride of the staged heights: odd, so that the column reads of
// the range pass hit distinct banks
__host__ __device__ __forceinline__ int surface_stride(int T) { return T | 1; }
// 32-bit words of a line mask: the cells' bits and 64 zero bits on each side;
// odd, so that the lanes of a wave reading one word of many lines hit
// distinct banks (as the strides below)
__host__ __device__ __forceinline__ int surface_mask_stride(int T) {
  return 2 * ((T + 63) >> 6) + 5;
}
// Distances are kept line-fastest, [tile column][line], so that the rings of a
// cone are consecutive bytes.  Ring lookups run up to seven rings past D, in
// whole words: bytes on each side of the lines, which hold "none" (the lookup
// subtracts whole words, so every byte it reads has to be below 128).
constexpr int kSurfPad = 12;
__host__ __device__ __forceinline__ int surface_dist_stride(int T) {
  return 4 * (((T + 2 * kSurfPad + 3) >> 2) | 1);
}

// 32 bits of a bit string starting at bit s.
__device__ __forceinline__ uint32_t bits_at(const uint32_t* w, int s) {
  const int i = s >> 5;
  return __builtin_amdgcn_alignbit(w[i + 1], w[i], (uint32_t)s & 31u);
}

// Distance from cell k of a line mask to its nearest set bit; kSurfNone where
// there is none within 31 (within 64 with FAR) cells.
constexpr uint32_t kSurfNone = 127;
template <bool FAR>
__device__ __forceinline__ uint32_t line_distance(const uint32_t* m, int k) {
  const uint32_t* w = m + (k >> 5);
  const uint32_t sh = (uint32_t)k & 31u;
  // cells k-32..k-1 (bit 31 = k-1) and k..k+31 (bit 0 = k)
  const uint32_t lo = __builtin_amdgcn_alignbit(w[2], w[1], sh);
  const uint32_t hi = __builtin_amdgcn_alignbit(w[3], w[2], sh);
  uint32_t a = lo ? (uint32_t)__builtin_clz(lo) + 1u : kSurfNone;
  uint32_t b = hi ? (uint32_t)__builtin_ctz(hi) : kSurfNone;
  if (FAR) {  // cells k-64..k-33 and k+32..k+63, and k+64
    const uint32_t lo2 = __builtin_amdgcn_alignbit(w[1], w[0], sh);
    const uint32_t hi2 = __builtin_amdgcn_alignbit(w[4], w[3], sh);
    const uint32_t a2 = lo2 ? (uint32_t)__builtin_clz(lo2) + 33u : kSurfNone;
    const uint32_t b2 = hi2 ? (uint32_t)__builtin_ctz(hi2) + 32u
                            : ((w[4] >> sh) & 1u ? 64u : kSurfNone);
    a = min(a, a2);
    b = min(b, b2);
  }
  return min(a, b);
}

// Normal equations of the N x N window of a defined pixel (heights relative
// to the centre's).
struct PlaneSums {
  int32_t n, sx, sy, sxx, syy, sxy;
  int64_t sz, sxz, syz, szz;
};

__device__ __forceinline__ void plane_sums(const int32_t* c, const int TS, const int h,
                                           const int32_t hc, PlaneSums& s) {
  s = {};
  for (int dx = -h; dx <= h; dx++)
    for (int dy = -h; dy <= h; dy++) {
      const int32_t v = c[dx * TS + dy];
      if (v == INT32_MIN) continue;
      const int64_t dz = (int64_t)v - hc;
      s.n++;
      s.sx += dx;
      s.sy += dy;
      s.sxx += dx * dx;
      s.syy += dy * dy;
      s.sxy += dx * dy;
      s.sz += dz;
      s.sxz += dx * dz;
      s.syz += dy * dz;
      s.szz += dz * dz;
    }
}

// The same for N = 5 and heights within 2^23 of each other (the first moments
// stay below 30 * 2^23, so 32-bit sums are exact).  The counts are summed as
// packed byte fields, offsets making every field non-negative: a row's
// n | sum(dy+2) << 8 | sum(dy^2) << 16, then over the rows their sums (at most
// 25, 50, 50), the sums weighted by dx+2 (at most 50, 100) and by dx^2 (50).
__device__ __forceinline__ void plane_sums5(const int32_t* c, const int TS, const int32_t hc,
                                            PlaneSums& s) {
  uint32_t c0 = 0, c1 = 0, c2 = 0;
  int32_t sz = 0, sxz = 0, syz = 0;
  int64_t szz = 0;
#pragma unroll
  for (int dx = -2; dx <= 2; dx++) {
    uint32_t r = 0;
    int32_t rz = 0;
#pragma unroll
    for (int dy = -2; dy <= 2; dy++) {
      const int32_t v = c[dx * TS + dy];
      const bool def = v != INT32_MIN;
      const int32_t dz = def ? v - hc : 0;
      r += def ? 1u | (uint32_t)(dy + 2) << 8 | (uint32_t)(dy * dy) << 16 : 0u;
      rz += dz;
      syz += dy * dz;
      szz += (int64_t)dz * dz;
    }
    c0 += r;
    c1 += r * (uint32_t)(dx + 2);
    c2 += (r & 0xFFu) * (uint32_t)(dx * dx);
    sz += rz;
    sxz += dx * rz;
  }
  s.n = (int32_t)(c0 & 0xFFu);
  s.sy = (int32_t)((c0 >> 8) & 0xFFu) - 2 * s.n;
  s.syy = (int32_t)(c0 >> 16);
  s.sx = (int32_t)(c1 & 0xFFu) - 2 * s.n;
  s.sxx = (int32_t)c2;
  // sum (dx+2)(dy+2) = sxy + 2 sx + 2 sy + 4 n
  s.sxy = (int32_t)((c1 >> 8) & 0xFFu) - 2 * (s.sx + s.sy) - 4 * s.n;
  s.sz = sz;
  s.sxz = sxz;
  s.syz = syz;
  s.szz = szz;
}

// Least-squares plane from the sums; I = integer type that holds the
// determinant's terms (int32 for N = 5: at most 25 * 50 * 50 * 3, with factors
// of at most 24 bits).
__device__ __forceinline__ int32_t mul_i(int32_t a, int32_t b) { return __mul24(a, b); }
__device__ __forceinline__ int64_t mul_i(int64_t a, int64_t b) { return a * b; }

template <class I>
__device__ __forceinline__ bool plane_solve(const PlaneSums& s, const double q2m, float& slope,
                                            float& rough) {
  const I n = s.n, sx = s.sx, sy = s.sy, sxx = s.sxx, syy = s.syy, sxy = s.sxy;
  // adjugate of M = [[sxx sxy sx] [sxy syy sy] [sx sy n]] (symmetric)
  const I c00 = mul_i(syy, n) - mul_i(sy, sy);
  const I c01 = mul_i(sy, sx) - mul_i(sxy, n);
  const I c02 = mul_i(sxy, sy) - mul_i(syy, sx);
  const I c11 = mul_i(sxx, n) - mul_i(sx, sx);
  const I c12 = mul_i(sxy, sx) - mul_i(sxx, sy);
  const I c22 = mul_i(sxx, syy) - mul_i(sxy, sxy);
  const I det = mul_i(sxx, c00) + mul_i(sxy, c01) + mul_i(sx, c02);
  if (n < 3 || det == 0) return false;
  const double inv = 1.0 / (double)det;
  const double bx = (double)s.sxz, by = (double)s.syz, bz = (double)s.sz;
  const double al = ((double)c00 * bx + (double)c01 * by + (double)c02 * bz) * inv;
  const double be = ((double)c01 * bx + (double)c11 * by + (double)c12 * bz) * inv;
  const double ga = ((double)c02 * bx + (double)c12 * by + (double)c22 * bz) * inv;
  // residual sum of squares of the least-squares plane: z.z - beta.(X^T z)
  // (integer sums exact; |dz| < 2^23 Q units as nz <= 128, so the double
  // cancellation error stays far below the roughness tolerance)
  const double ss = fmax((double)s.szz - (al * bx + be * by + ga * bz), 0.0);
  slope = (float)(sqrt(al * al + be * be) / 65536.0);
  rough = (float)(ss / (double)n * q2m * q2m);
  return true;
}

// Stages the tile's heights row by row (a wave per row, lanes along y).  A
// wave issues the loads of ROWS rows before it stores any (addresses clamped
// into the map, so every load is in bounds; with EDGE the tile reaches past
// the map and cells outside it take the empty value).
template <int MW, int ROWS, int WAVES, bool EDGE>
__device__ __forceinline__ void surface_stage(const SurfaceArgs& a, const int T, const int TS,
                                              const int gx0, const int gy0, int32_t* th) {
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  int gy[MW];
#pragma unroll
  for (int w = 0; w < MW; w++) gy[w] = min(max(gy0 + 64 * w + lane, 0), a.ny - 1);
  for (int r0 = wv; r0 < T; r0 += ROWS * WAVES) {
    int32_t v[ROWS][MW];
#pragma unroll
    for (int j = 0; j < ROWS; j++) {
      const int32_t* row = a.hq + (int64_t)min(max(gx0 + r0 + j * WAVES, 0), a.nx - 1) * a.ny;
#pragma unroll
      for (int w = 0; w < MW; w++) v[j][w] = row[gy[w]];
    }
#pragma unroll
    for (int j = 0; j < ROWS; j++) {
      const int r = r0 + j * WAVES;
      if (r >= T) break;
      const int gx = gx0 + r;
#pragma unroll
      for (int w = 0; w < MW; w++) {
        const int k = 64 * w + lane;
        const bool in = !EDGE || (gx >= 0 && gx < a.nx && gy0 + k == gy[w]);
        if (k < T) th[r * TS + k] = in ? v[j][w] : INT32_MIN;
      }
    }
  }
}

template <int WAVES, bool EDGE>
__device__ __forceinline__ void surface_stage_w(const SurfaceArgs& a, const int T, const int TS,
                                                const int gx0, const int gy0, int32_t* th) {
  if (T <= 64) surface_stage<1, 4, WAVES, EDGE>(a, T, TS, gx0, gy0, th);
  else if (T <= 128) surface_stage<2, 6, WAVES, EDGE>(a, T, TS, gx0, gy0, th);
  else surface_stage<3, 5, WAVES, EDGE>(a, T, TS, gx0, gy0, th);
}

// The staged rows' masks from the column pass's bits (bit c of the bit string
// = pixel c defined); cells outside the map are clear.
template <int NT>
__device__ __forceinline__ void surface_row_masks(const SurfaceArgs& a, const int T, const int MS,
                                                  const int gx0, const int gy0, uint32_t* rmask) {
  const int words = 2 * ((T + 63) >> 6);
  const int last = ((a.nx * a.ny + 63) >> 6) * 2 - 1;  // words of the bit string - 1
  for (int i = threadIdx.x; i < T * words; i += NT) {
    const int r = i / words, w = i - r * words;
    const int gx = gx0 + r, y0 = gy0 + 32 * w;  // cells y0 .. y0 + 31 of map row gx
    uint32_t v = 0;
    if (gx >= 0 && gx < a.nx && y0 + 31 >= 0 && y0 < a.ny) {
      const int s = gx * a.ny + y0;  // may start before the bit string
      const int q = s >> 5;
      v = __builtin_amdgcn_alignbit(a.defbits[min(q + 1, last)], a.defbits[max(q, 0)],
                                    (uint32_t)s & 31u);
      if (y0 < 0) v &= ~0u << -y0;
      const int n = min(a.ny - y0, T - 32 * w);  // cells of the word in the map and the tile
      if (n < 32) v &= n > 0 ? (1u << n) - 1u : 0u;
    }
    rmask[r * MS + 2 + w] = v;
  }
}

// Distances of every line at the tile's columns (col 0: rows; 1: columns),
// four lines per thread.
template <bool FAR, int TILE, int NT>
__device__ __forceinline__ void surface_distances(const uint32_t* rmask, const uint32_t* cmask,
                                                  const int MS, const int T, const int H,
                                                  uint8_t* rdist, uint8_t* cdist, const int DS) {
  const int nq = (T + 3) >> 2, nw = DS >> 2;
  for (int i = threadIdx.x; i < 2 * TILE * nw; i += NT) {
    const int jj = i / nw, q = i - jj * nw - kSurfPad / 4;
    const bool col = jj >= TILE;
    const int j = col ? jj - TILE : jj;
    const uint32_t* m = col ? cmask : rmask;
    uint32_t v = 0;
    if (q < 0 || q >= nq) v = kSurfNone * 0x01010101u;
    else
#pragma unroll
    for (int e = 0; e < 4; e++)
      v |= line_distance<FAR>(m + min(4 * q + e, T - 1) * MS, H + j) << (8 * e);
    *(uint32_t*)((col ? cdist : rdist) + j * DS + 4 * q) = v;
  }
}

// Range of the defined cells of up to four slices: window 2k (2k + 1) holds
// the bits of slice k's cells from cell[2k] (cell[2k + 1]) on, a word address
// of th, consecutive cells 1 (k < 2) or TS words apart.  The eight windows
// advance together, one cell each per round, so that their LDS reads overlap;
// an empty window reads its last cell again, or another window's.
__device__ __forceinline__ void slice_cells(const int32_t* th, const int cell[8], const int TS,
                                            uint32_t win[8], int32_t& lo, int32_t& hi) {
  int at[8], any = 0;
#pragma unroll
  for (int k = 0; k < 8; k++) any = win[k] ? cell[k] + __mul24(__builtin_ctz(win[k]), k < 4 ? 1 : TS) : any;
#pragma unroll
  for (int k = 0; k < 8; k++) at[k] = any;
  while ((win[0] | win[1] | win[2]) | (win[3] | win[4] | win[5]) | (win[6] | win[7])) {
    int32_t v[8];
#pragma unroll
    for (int k = 0; k < 8; k++) {
      const int i = __ffs(win[k]) - 1;
      at[k] = win[k] ? cell[k] + (k < 4 ? i : __mul24(i, TS)) : at[k];
      v[k] = th[at[k]];
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
      lo = min(lo, v[k]);
      hi = max(hi, v[k]);
      win[k] &= win[k] - 1u;
    }
  }
}

// Spread (maximum - minimum) of the heights of the defined cells in the
// stopping slices of the four cones of the undefined pixel at staged (tx, ty);
// -1 without any.  rd, cd: its line distances (rows at its column, columns at
// its row), pointing at its own line.
__device__ __forceinline__ int64_t cone_spread(const int32_t* th, const uint32_t* rmask,
                                               const uint32_t* cmask, const uint8_t* rd,
                                               const uint8_t* cd, const int32_t* lds, const int TS,
                                               const int MS, const int tx, const int ty,
                                               const int D) {
  // cones 0/1: +x/-x (slices on staged rows), 2/3: +y/-y (staged columns);
  // first[k]: first ring holding a defined cell.  Eight rings of every cone
  // per round, as aligned words shifted to the ring's byte (rings past D
  // are read from the free bytes or other lines and rejected below: the
  // first ring found is the smallest).
  int wi[4];
  uint32_t sh[4];
#pragma unroll
  for (int k = 0; k < 4; k++) {
    // byte offset of the lowest ring byte of the first round
    const uint32_t o = (uint32_t)((k < 2 ? rd : cd) - (const uint8_t*)lds) + (k & 1 ? -8 : 1);
    wi[k] = (int)(o >> 2);
    sh[k] = o & 3u;
  }
  // A ring holds a defined cell iff its byte is at most the ring number: with
  // both below 128, bit 7 of 128 + ring - byte.  hit / at: the bits of the
  // first four rings with one, and the lowest of those rings.
  uint32_t hit[4] = {0, 0, 0, 0};
  int at[4] = {0, 0, 0, 0};
  for (int d = 1, w = 0; d <= D; d += 8, w += 2) {
    uint32_t v[4][3];
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
      for (int e = 0; e < 3; e++) v[k][e] = (uint32_t)lds[wi[k] + (k & 1 ? -w : w) + e];
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const bool down = k & 1;  // ring numbers fall with the byte address
      const uint32_t ramp = (uint32_t)d * 0x01010101u + (down ? 0x80818283u : 0x83828180u);
      const uint32_t b0 = __builtin_amdgcn_alignbyte(v[k][1], v[k][0], sh[k]);
      const uint32_t b1 = __builtin_amdgcn_alignbyte(v[k][2], v[k][1], sh[k]);
      const uint32_t mn = (ramp - (down ? b1 : b0)) & 0x80808080u;
      const uint32_t mf = (ramp + 0x04040404u - (down ? b0 : b1)) & 0x80808080u;
      const bool open = hit[k] == 0;
      at[k] = open ? (mn ? d : d + 4) : at[k];
      hit[k] = open ? (mn ? mn : mf) : hit[k];
    }
    if (min(min(hit[0], hit[1]), min(hit[2], hit[3])) != 0) break;
  }
  int first[4];
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int e = (k & 1 ? __builtin_clz(hit[k] | 1u) : __builtin_ctz(hit[k] | 0x80000000u)) >> 3;
    first[k] = hit[k] ? at[k] + e : 255;
  }
  // the slices' cells: offsets -31..0 and 1..32 from the centre
  int32_t lo = INT32_MAX, hi = INT32_MIN;
  uint32_t win[8];
  int cell[8];
  bool wide = false;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int d = first[k];
    const bool ok = d <= D;
    const int dc = ok ? d : 0;
    const int line = (k < 2 ? tx : ty) + (k & 1 ? -dc : dc), oth = k < 2 ? ty : tx;
    const uint32_t* m = (k < 2 ? rmask : cmask) + __mul24(line, MS);
    const uint32_t wl = bits_at(m, oth + 33), wr = bits_at(m, oth + 65);
    const int dl = min(dc, 31);
    win[2 * k] = ok ? wl & (~0u << (31 - dl)) : 0u;
    win[2 * k + 1] = ok ? wr & (0x7FFFFFFFu >> (31 - dl)) : 0u;
    const int mid = k < 2 ? __mul24(line, TS) + oth : __mul24(oth, TS) + line;
    cell[2 * k] = mid - 31 * (k < 2 ? 1 : TS);
    cell[2 * k + 1] = mid + (k < 2 ? 1 : TS);
    wide |= ok & (d > 31);
  }
  slice_cells(th, cell, TS, win, lo, hi);
  if (wide) {
    // slices of rings past 31: offsets -63..-32 and 32..63, and +-64
#pragma unroll
    for (int k = 0; k < 4; k++) {
      const int d = first[k];
      const bool ok = d <= D && d > 31;
      const int st = k < 2 ? 1 : TS;
      const int line = (k < 2 ? tx : ty) + (k & 1 ? -d : d), oth = k < 2 ? ty : tx;
      const int lc = ok ? line : 0;
      const uint32_t* m = (k < 2 ? rmask : cmask) + __mul24(lc, MS);
      const int dw = ok ? min(d, 63) : 32;
      win[2 * k] = ok ? bits_at(m, oth + 1) & (~0u << (63 - dw)) : 0u;
      win[2 * k + 1] = ok ? bits_at(m, oth + 96) & (~0u >> (63 - dw)) : 0u;
      const int mid = k < 2 ? __mul24(lc, TS) + oth : __mul24(oth, TS) + lc;
      cell[2 * k] = mid - 63 * st;
      cell[2 * k + 1] = mid + 32 * st;
      if (ok && d == 64) {
#pragma unroll
        for (int e = -64; e <= 64; e += 128) {
          const int32_t v = th[mid + e * st];
          if (v != INT32_MIN) {
            lo = min(lo, v);
            hi = max(hi, v);
          }
        }
      }
    }
    slice_cells(th, cell, TS, win, lo, hi);
  }
  return hi == INT32_MIN ? -1 : (int64_t)hi - lo;
}

template <int NT, int TILE>
__device__ __forceinline__ void surface_body(const SurfaceArgs& a, const bool wild, const int H,
                                             const int bx, const int by) {
  constexpr int kPix = TILE * TILE;  // tile pixels
  constexpr int kWaves = NT / 64;    // waves of the block
  constexpr int kPer = kPix > NT ? kPix / NT : 1;  // tile pixels per thread
  static_assert(kPix % 64 == 0 && NT % 64 == 0 && (kPix <= NT || kPer * NT == kPix), "whole waves");
  static_assert(kWaves <= 16, "one entry per lane of a row");
  extern __shared__ __attribute__((aligned(16))) int32_t lds[];
  const int T = TILE + 2 * H;           // staged tile edge
  const int TS = surface_stride(T);     // LDS row stride of th
  const int MS = surface_mask_stride(T);
  const int DS = surface_dist_stride(T);
  int32_t* th = lds;                                            // [T][TS]
  uint32_t* rmask = (uint32_t*)(lds + T * TS);                  // [T][MS]
  uint32_t* cmask = rmask + T * MS;                             // [T][MS]
  uint8_t* rdist = (uint8_t*)(cmask + T * MS) + kSurfPad;       // [TILE][DS]: tile column, row
  uint8_t* cdist = rdist + TILE * DS;                           // [TILE][DS]: tile row, column
  int16_t* order = (int16_t*)(cdist + TILE * DS - kSurfPad);    // [kPix]
  const int gx0 = bx * TILE - H, gy0 = by * TILE - H;
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  const int h = a.half_fit, D = a.search_d;

  // ---- heights and row masks
  if (gx0 >= 0 && gy0 >= 0 && gx0 + T <= a.nx && gy0 + T <= a.ny)
    surface_stage_w<kWaves, false>(a, T, TS, gx0, gy0, th);
  else
    surface_stage_w<kWaves, true>(a, T, TS, gx0, gy0, th);
  surface_row_masks<NT>(a, T, MS, gx0, gy0, rmask);
  for (int i = threadIdx.x; i < 2 * T; i += NT) {  // the masks' zero ends
    uint32_t* m = rmask + i * MS;  // cmask follows rmask
    m[0] = m[1] = m[MS - 3] = m[MS - 2] = 0u;
  }
  __syncthreads();

  // ---- pixel order: defined pixels (plane fit) and undefined ones (cone
  // search) go to separate waves, listed defined-first.  Lane l counts tile
  // row l; counts of defined | undefined << 16.
  int nd, nu;
  {
    const int vy = min(TILE, a.ny - by * TILE);
    const auto row_bits = [&](int row, unsigned long long& def, unsigned long long& und) {
      const unsigned long long m = bx * TILE + row < a.nx ? ~0ull >> (64 - vy) : 0ull;
      const uint32_t* w = rmask + (H + row) * MS;
      def = bits_at(w, H + 64);
      if (TILE == 64) def |= (unsigned long long)bits_at(w, H + 96) << 32;
      def &= m;
      und = ~def & m;
    };
    unsigned long long def, und;
    row_bits(lane & (TILE - 1), def, und);
    const int cnt = __popcll(def) | __popcll(und) << 16;
    int x = cnt;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, true);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, true);
    if (TILE >= 32) {
      const int t0 = __builtin_amdgcn_readlane(x, 15);
      const int t1 = TILE == 64 ? t0 + __builtin_amdgcn_readlane(x, 31) : 0;
      const int t2 = TILE == 64 ? t1 + __builtin_amdgcn_readlane(x, 47) : 0;
      const int q = (lane & (TILE - 1)) >> 4;
      x += q == 0 ? 0 : q == 1 ? t0 : q == 2 ? t1 : t2;
    }
    const int tot = __builtin_amdgcn_readlane(x, TILE - 1);
    nd = tot & 0xFFFF;
    nu = tot >> 16;
#pragma unroll
    for (int k = 0; k < kPer; k++) {
      const int p = k * NT + threadIdx.x, row = p / TILE, col = p - row * TILE;
      if (kPix < NT && p >= kPix) break;  // whole waves
      const int before = __shfl(x - cnt, row);
      row_bits(row, def, und);
      const unsigned long long below = (1ull << col) - 1ull;
      if ((def >> col) & 1u) order[(before & 0xFFFF) + __popcll(def & below)] = (int16_t)p;
      if ((und >> col) & 1u) order[kPix - 1 - ((before >> 16) + __popcll(und & below))] = (int16_t)p;
    }
  }
  if (nu) {
    // column masks: lane = row, a ballot per column; a wave takes kChunk
    // consecutive columns, whose bits are one word of each row
    constexpr int kChunk = 6;
    for (int w = 0; w < (T + 63) >> 6; w++) {
      const int r = 64 * w + lane;
      for (int c0 = wv * kChunk; c0 < T; c0 += kWaves * kChunk) {
        const uint32_t v = r < T ? bits_at(rmask + r * MS, 64 + c0) : 0u;
        uint32_t mword = 0;
#pragma unroll
        for (int e = 0; e < kChunk; e++) {
          const unsigned long long b = __ballot((v >> e) & 1u);
          mword = lane == 2 * e ? (uint32_t)b : mword;
          mword = lane == 2 * e + 1 ? (uint32_t)(b >> 32) : mword;
        }
        const int c = c0 + (lane >> 1);
        if (lane < 2 * kChunk && c < T) cmask[c * MS + 2 + 2 * w + (lane & 1)] = mword;
      }
    }
    __syncthreads();
    if (D <= 31) surface_distances<false, TILE, NT>(rmask, cmask, MS, T, H, rdist, cdist, DS);
    else surface_distances<true, TILE, NT>(rmask, cmask, MS, T, H, rdist, cdist, DS);
  }
  __syncthreads();

  // ---- slots [0, nd): defined pixels, [kPix - nu, kPix): undefined
#pragma unroll 1
  for (int k = 0; k < kPer; k++) {
    const int slot = k * NT + threadIdx.x;
    if (slot >= kPix || (slot >= nd && slot < kPix - nu)) continue;
    const int me = order[slot];
    const int px = me / TILE, py = me - px * TILE;
    const int tx = px + H, ty = py + H;
    const int64_t c = (int64_t)(bx * TILE + px) * a.ny + by * TILE + py;
    uint8_t fl = a.flags[c];
    float slope = __uint_as_float(kQNaN), rough = __uint_as_float(kQNaN);
    if (slot < nd) {
      const int32_t* tc = th + tx * TS + ty;
      PlaneSums s;
      bool ok;
      if (h == 2 && !wild) {
        plane_sums5(tc, TS, *tc, s);
        ok = plane_solve<int32_t>(s, a.q2m, slope, rough);
      } else {
        plane_sums(tc, TS, h, *tc, s);
        ok = plane_solve<int64_t>(s, a.q2m, slope, rough);
      }
      if (ok) fl |= 32;
    } else {
      if (cone_spread(th, rmask, cmask, rdist + py * DS + tx, cdist + px * DS + ty, lds, TS, MS, tx,
                      ty, D) > a.tau_q)
        fl |= 16;
    }
    a.slope[c] = slope;
    a.rough[c] = rough;
    a.flags[c] = fl;
  }
}


// Lookup-table export.  Ranks follow window-local column order: pass 1 gives
// every local column its occupied-voxel count prefix within its group of 64
// columns and each group its count, pass 2 sums the counts of every super
// group of 64 groups (and makes them prefixes within it), pass 3 writes the
// table and the data array region by region, scanning the sums of the super
// groups in a wave (many of them are scanned once before, see kWaveSupers).
// After a 2D export the first two passes are already done, by its column pass and
// by one wave in each of the first blocks of its surface pass: a scan of all groups
// in a launch of its own took 5 us at 4,096 groups and 20 us at 16,384, and a
// block more in the surface pass 7 us (a compute unit with two of its blocks).
constexpr int kGroup = 64;

__device__ __forceinline__ void lut_count_body(const LutArgs& a, const int blk) {
  const int nx = a.d.nx, ny = a.d.ny;
  const int lane = __lane_id();
  const int c = blk * kBlock + threadIdx.x;
  int cnt = 0;
  if (c < nx * ny) {
    const int x = c / ny, y = c - x * ny;
    const int64_t scol = (int64_t)wrap_add(x + a.d.ro[0], nx) * ny + wrap_add(y + a.d.ro[1], ny);
    cnt = __popcll(a.occ[scol * a.d.W]);
    if (a.d.W > 1) cnt += __popcll(a.occ[scol * a.d.W + 1]);
  }
  const int incl = wave_scan(cnt);
  if (c < nx * ny) a.colpre[c] = incl - cnt;
  const int g = c >> 6;
  if (lane == 63 && g * kGroup < nx * ny) a.group_cnt[g] = incl;
}


// Pass 2: the counts of super group g become exclusive prefixes within it, and
// sum[g] their sum, by one wave.
__device__ __forceinline__ void super_sum_body(int32_t* cnt, const int n, int32_t* sum,
                                               const int g) {
  const int i = 64 * g + __lane_id();
  const int v = i < n ? cnt[i] : 0;
  const int s = wave_scan(v);
  if (i < n) cnt[i] = s - v;
  if (__lane_id() == 63) sum[g] = s;
}

// Exclusive prefix of base[0..nb) in place (one block); *n_occupied = the sum.
template <int NT>
__device__ __forceinline__ void lut_scan_body(int32_t* base, const int nb, int64_t* n_occupied) {
  __shared__ int64_t wsum[NT / 64];
  const int t = threadIdx.x;
  const int per = (nb + NT - 1) / NT;
  const int b0 = min(t * per, nb), b1 = min(b0 + per, nb);
  // the thread's counts in chunks of 8 loads in flight (clamped in-bounds
  // loads, masked sums); the first chunk stays in registers for the writes
  constexpr int kChunk = 8;
  int32_t v0[kChunk];
  int64_t s = 0;
  for (int c = b0; c < b1; c += kChunk) {
    int32_t v[kChunk];
#pragma unroll
    for (int k = 0; k < kChunk; k++) v[k] = base[min(c + k, nb - 1)];
#pragma unroll
    for (int k = 0; k < kChunk; k++) {
      if (c + k < b1) s += v[k];
      if (c == b0) v0[k] = v[k];
    }
  }
  const int lane = __lane_id(), w = t >> 6;
  int64_t v = s;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int64_t u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  if (lane == 63) wsum[w] = v;
  __syncthreads();
  if (t == 0) {
    int64_t acc = 0;
    for (int k = 0; k < NT / 64; k++) {
      const int64_t q = wsum[k];
      wsum[k] = acc;
      acc += q;
    }
    *n_occupied = acc;
  }
  __syncthreads();
  int64_t run = wsum[w] + v - s;  // exclusive prefix of this thread's range
#pragma unroll
  for (int k = 0; k < kChunk; k++) {
    if (b0 + k < b1) {
      base[b0 + k] = (int32_t)run;
      run += v0[k];
    }
  }
  for (int b = b0 + kChunk; b < b1; b++) {
    const int32_t q = base[b];
    base[b] = (int32_t)run;
    run += q;
  }
}


// ---- storage regions: 4 x 16 columns (four 4 x 4 bricks, contiguous in
// memory).  The kernels that turn the whole map between storage order and
// window-local order (the table, density and feature exports, the import)
// take one region per block: the passes (or table entries) go through LDS
// rows in window-local z order, so that both sides are read and written in
// 16-byte words; hits and lowest returns, which only occupied voxels have, are
// touched one voxel at a time where the occupancy words say so.
constexpr int kRegCols = 64;
constexpr int kLutLoads = 4;  // 16-byte region loads per thread per batch

// LDS row stride of a column's passes: a multiple of 4 words.
__host__ __device__ __forceinline__ int lut_row(int nz) { return ((nz + 3) & ~3) + 4; }

// The columns of a region (slot t = 16 ix + 4 b + iy: brick b, column (ix, iy)
// of the brick): occupancy in window-local z order, storage index of z = 0,
// window-local column index (-1 outside the map) and prefix of the occupied
// voxels in slot order.
struct RegionCols {
  unsigned long long lo[kRegCols], hi[kRegCols];
  int32_t base[kRegCols], col[kRegCols], pre[kRegCols + 1];
};

__device__ __forceinline__ int32_t region_col(const Dims& d, const int bxr, const int byr,
                                              const int t, int& sx, int& sy) {
  sx = 4 * bxr + (t >> 4);
  sy = 16 * byr + (t & 15);
  if (sx >= d.nx || sy >= d.ny) return -1;
  const int x = sx - d.ro[0] + (sx < d.ro[0] ? d.nx : 0);
  const int y = sy - d.ro[1] + (sy < d.ro[1] ? d.ny : 0);
  return x * d.ny + y;
}

// 16-byte word k4 of a region holds brick b, level zs, brick row iy
// (k4 = 4 (b nz + zs) + iy), voxels ix = 0..3; slot of voxel ix = 16 ix + 4 b + iy.
__device__ __forceinline__ int region_word(const int k4, const int nz, const uint32_t nz_magic,
                                           int& zs) {
  const int bz = k4 >> 2, iy = k4 & 3;
  const int b = nz == 1 ? bz : (int)__umulhi((uint32_t)bz, nz_magic);
  zs = bz - b * nz;
  return 4 * b + iy;
}

// Loads the passes of region (bxr, byr) into the LDS rows and describes its
// columns (wave 0, while the first loads are in flight; extra(t, c) for slot t
// = window-local column c, -1 outside the map, called by the whole wave).  Ends
// without a barrier.
template <class Extra>
__device__ __forceinline__ void region_load(const Dims& d, const int32_t* passes,
                                            const unsigned long long* occ, const uint32_t nz_magic,
                                            const int bxr, const int byr, int32_t* lpass,
                                            RegionCols& rc, Extra extra) {
  const int nz = d.nz, roz = d.ro[2], nzp = lut_row(nz);
  const int tid = threadIdx.x;
  const int nv4 = min(4, d.nby - 4 * byr) * nz * 4;
  const int4* __restrict__ src = (const int4*)(passes + col_base(d, 4 * bxr, 16 * byr));
  for (int k0 = 0; k0 < nv4; k0 += kLutLoads * kBlock) {
    int4 v[kLutLoads];
#pragma unroll
    for (int u = 0; u < kLutLoads; u++) {
      // clamped, not skipped: every lane loads (in bounds), the stores below
      // skip the words past the region
      v[u] = src[min(k0 + u * kBlock + tid, nv4 - 1)];
    }
    if (k0 == 0 && tid < kRegCols) {
      int sx, sy;
      const int32_t c = region_col(d, bxr, byr, tid, sx, sy);
      // the occupancy words and extra()'s loads in one round trip: the words
      // are loaded first (from a clamped column) and used last
      const int64_t ow = c >= 0 ? ((int64_t)sx * d.ny + sy) * d.W : 0;
      const unsigned long long w0 = occ[ow], w1 = occ[ow + d.W - 1];
      extra(tid, c);
      const Mask128 m = c >= 0 ? rotate_mask(w0, d.W > 1 ? w1 : 0ull, nz, roz) : Mask128{0ull, 0ull};
      const int cnt = __popcll(m.lo) + __popcll(m.hi);
      const int incl = wave_scan(cnt);
      rc.lo[tid] = m.lo;
      rc.hi[tid] = m.hi;
      rc.base[tid] = col_base(d, sx, sy);
      rc.col[tid] = c;
      rc.pre[tid] = incl - cnt;
      if (tid == kRegCols - 1) rc.pre[kRegCols] = incl;
    }
#pragma unroll
    for (int u = 0; u < kLutLoads; u++) {
      const int k4 = k0 + u * kBlock + tid;
      if (k4 < nv4) {
        int zs;
        const int t = region_word(k4, nz, nz_magic, zs);
        const int lz = zs >= roz ? zs - roz : zs - roz + nz;
        int32_t* row = lpass + t * nzp + lz;
        row[0] = v[u].x;
        row[16 * nzp] = v[u].y;
        row[32 * nzp] = v[u].z;
        row[48 * nzp] = v[u].w;
      }
    }
  }
}

// Occupied voxel o of a region (o < rc.pre[kRegCols]): its slot (the one with
// pre[t] <= o < pre[t + 1]) and number r within its column; its level is the
// set bit of rank r.
__device__ __forceinline__ int region_voxel(const RegionCols& rc, const int o, int& r, int& z) {
  int t = 0;
#pragma unroll
  for (int step = kRegCols / 2; step >= 1; step >>= 1)
    if (rc.pre[t + step] <= o) t += step;
  r = o - rc.pre[t];
  z = select_bit(Mask128{rc.lo[t], rc.hi[t]}, r);
  return t;
}

// Calls item(t, q) for the quads q (window-local z = 4q .. 4q + 3) of every
// column of the region inside the map; quads per column rounded up to a power
// of two so that t and q are shifts.
template <class Item>
__device__ __forceinline__ void region_quads(const RegionCols& rc, const int nz, Item item) {
  const int nq = (nz + 3) >> 2;
  const int qsh = nq > 1 ? 32 - __clz(nq - 1) : 0;
  for (int i = threadIdx.x; i < (kRegCols << qsh); i += kBlock) {
    const int t = i >> qsh, q = i & ((1 << qsh) - 1);
    if (q < nq && rc.col[t] >= 0) item(t, q);
  }
}

// Four consecutive words of the output, streaming (written once, not read back).
template <class T>
__device__ __forceinline__ void store_quad(T* out, const T v[4], const int n, const bool vec) {
  typedef T v4t __attribute__((ext_vector_type(4)));
  if (vec) {
    const v4t vv = {v[0], v[1], v[2], v[3]};
    __builtin_nontemporal_store(vv, (v4t*)out);
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (e < n) __builtin_nontemporal_store(v[e], out + e);
  }
}

// Pass 3: the table, and the records of the occupied voxels one thread per
// voxel (every gather issued at once).
__device__ __forceinline__ void lut_write_body(const LutArgs& a, const uint32_t nz_magic,
                                               const int bxr, const int byr) {
  extern __shared__ __attribute__((aligned(16))) int32_t lpass[];  // [64][lut_row(nz)]
  __shared__ RegionCols rc;
  __shared__ int32_t sbase[kRegCols];  // rank of the column's first occupied voxel
  const int nz = a.d.nz, roz = a.d.ro[2], nzp = lut_row(nz);
  region_load(a.d, a.passes, a.occ, nz_magic, bxr, byr, lpass, rc, [&](int t, int32_t c) {
    const int g = max(c, 0) >> 6, sg = g >> 6;
    const int32_t cp = a.colpre[max(c, 0)], gp = a.group_cnt[g];
    const int32_t s0 = a.super_sum[a.scanned ? sg : min(t, a.nsuper - 1)];
    int32_t base = c >= 0 ? cp + gp : 0;
    if (a.scanned) {
      base += s0;
    } else {  // at most kWaveSupers: a lane each
      const int v = t < a.nsuper ? s0 : 0;
      const int s = wave_scan(v);
      base += __shfl(s - v, sg);
      if (bxr == 0 && byr == 0 && t == 63) *a.n_occupied = s;
    }
    sbase[t] = base;
  });
  __syncthreads();
  const int nocc = rc.pre[kRegCols];
  for (int o = threadIdx.x; o < nocc; o += kBlock) {
    int r, z;
    const int t = region_voxel(rc, o, r, z);
    const int32_t rank = sbase[t] + r;
    if ((uint64_t)(int64_t)rank < (uint64_t)a.cap) {  // (0 <= rank < cap)
      const int64_t idx = rc.base[t] + ((int64_t)wrap_add(z + roz, nz) << 4);
      map_voxel_t d;
      d.hits = a.hits[idx];
      d.passes = lpass[t * nzp + z];
      d.min_qz = a.minqz[idx];
      a.data[rank] = d;
    }
  }
  const bool vec = (nz & 3) == 0 && ((uintptr_t)a.lut & 15) == 0;
  region_quads(rc, nz, [&](int t, int q) {
    const Mask128 mt = {rc.lo[t], rc.hi[t]};
    const int z0 = 4 * q;
    const int4 pv = *(const int4*)(lpass + t * nzp + z0);
    const int32_t p4[4] = {pv.x, pv.y, pv.z, pv.w};
    int32_t rank = sbase[t] + rank_below(mt, z0);
    int32_t v[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int z = z0 + e;
      const bool occ = z < nz && test_bit(mt, z);
      v[e] = occ ? rank : -1 - p4[e];
      rank += occ;
    }
    store_quad(a.lut + (int64_t)rc.col[t] * nz + z0, v, nz - z0, vec);
  });
}

}  // namespace
}  // namespace gvom
