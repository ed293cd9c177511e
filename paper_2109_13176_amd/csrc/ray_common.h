// Device helpers of the ray pass and the traversal: point
// transform and return, dominant axis, exact segment entry voxel and the
// exact integer voxel walk (Sec. III-C of arXiv 2109.13176).
#pragma once
#include <math.h>

#include "gvom_internal.h"

namespace gvom {
namespace {

__device__ __forceinline__ int32_t wrap_add(int32_t s, int32_t n) { return s >= n ? s - n : s; }

// Sums an int over the 64 lanes of the wave.
__device__ __forceinline__ int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

__device__ __forceinline__ int32_t mod_pos(int32_t v, int32_t n) {
  v %= n;
  return v < 0 ? v + n : v;
}

// x[k] for a lane-varying axis k, by selects (an indexed private array
// would go to scratch memory).
__device__ __forceinline__ int32_t sel3(const int k, const int32_t x0, const int32_t x1,
                                        const int32_t x2) {
  return k == 0 ? x0 : (k == 1 ? x1 : x2);
}

__device__ __forceinline__ int dominant_axis(const int32_t n[3]) {
  return (n[1] > n[0]) ? (n[2] > n[1] ? 2 : 1) : (n[2] > n[0] ? 2 : 0);
}

// Transform of point i (in firing order): q = Q16 world coordinates; f.hit is
// set when the return lies in the window.  Returns true when the ray can be
// traversed.
struct PointFlags {
  bool nonfinite = false, outrange = false, hit = false;
};

__device__ __forceinline__ bool point_pass(const InsertArgs& a, const int i, int32_t q[3],
                                           PointFlags& f) {
  q[0] = q[1] = q[2] = 0;
  if (i >= a.n) return false;
  int pidx = i;
  if (a.fw > 1) {
    const int b = i / a.azimuths;
    pidx = (i - b * a.azimuths) * a.fw + b;
  }
  const int32_t dims[3] = {a.d.nx, a.d.ny, a.d.nz};
  const float p0 = a.xyz[3 * pidx + 0];
  const float p1 = a.xyz[3 * pidx + 1];
  const float p2 = a.xyz[3 * pidx + 2];
  if (!(isfinite(p0) && isfinite(p1) && isfinite(p2))) {
    f.nonfinite = true;
    return false;
  }
  bool ok = true;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    float w = __builtin_fmaf(a.R[3 * k + 0], p0, a.t[k]);
    w = __builtin_fmaf(a.R[3 * k + 1], p1, w);
    w = __builtin_fmaf(a.R[3 * k + 2], p2, w);
    const float u = w * a.inv_r;
    const bool okk = isfinite(w) && fabsf(u) < 32768.0f;
    q[k] = okk ? (int32_t)floorf(u * 65536.0f) : 0;
    ok = ok && okk;
    const int64_t dd = (int64_t)q[k] - a.S[k];
    ok = ok && dd < (1 << 27) && -dd < (1 << 27);
  }
  if (!ok) {
    f.outrange = true;
    return false;
  }
  f.hit = true;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int32_t l = (q[k] >> 16) - a.O[k];
    f.hit = f.hit && l >= 0 && l < dims[k];
  }
  return true;
}

// The return of ray record {q, segments} (segments 0: no ray): f.e / f.ow /
// f.ob locate its voxel (storage index, occupancy word and bit).
struct Hit {
  bool on = false;
  int32_t e = 0;
  int64_t ow = 0;
  unsigned long long ob = 0;
};

__device__ __forceinline__ Hit find_hit(const InsertArgs& a, const int4 ray) {
  Hit f;
  const int32_t dims[3] = {a.d.nx, a.d.ny, a.d.nz};
  const int32_t l[3] = {(ray.x >> 16) - a.O[0], (ray.y >> 16) - a.O[1], (ray.z >> 16) - a.O[2]};
  f.on = ray.w > 0;
#pragma unroll
  for (int k = 0; k < 3; k++) f.on = f.on && l[k] >= 0 && l[k] < dims[k];
  if (f.on) {
    const int32_t ex = wrap_add(l[0] + a.d.ro[0], dims[0]);
    const int32_t ey = wrap_add(l[1] + a.d.ro[1], dims[1]);
    const int32_t ez = wrap_add(l[2] + a.d.ro[2], dims[2]);
    f.e = col_base(a.d, ex, ey) + (ez << 4);
    f.ow = (int64_t)(ex * dims[1] + ey) * a.d.W + (ez >> 6);
    f.ob = 1ull << (ez & 63);
  }
  return f;
}

// Recording a hit takes a count, a minimum and an or.  The minimum and the or
// only move one way, so a plain read that already satisfies the update makes
// that atomic unnecessary.  The reads are issued first (record_hit_issue) and
// the conditional atomics later (record_hit_finish), so their round trip can
// overlap other work of the caller; a stale read only costs a redundant
// atomic.
struct HitReads {
  int32_t mz = 0;
  unsigned long long ow = 0;
};

__device__ __forceinline__ HitReads record_hit_issue(const InsertArgs& a, const Hit& f) {
  HitReads r;
  if (f.on) {
    r.mz = a.minqz[f.e];
    r.ow = a.occ[f.ow];
    atomicAdd(&a.hits[f.e], 1);
  }
  return r;
}

__device__ __forceinline__ void record_hit_finish(const InsertArgs& a, const Hit& f,
                                                  const HitReads& r, const int32_t qz) {
  if (f.on) {
    if (qz < r.mz) atomicMin(&a.minqz[f.e], qz);
    if (!(r.ow & f.ob)) atomicOr(&a.occ[f.ow], f.ob);
  }
}

// With distinct counting: whether the hit is the first in its voxel this insert.
__device__ __forceinline__ int distinct_hit(const InsertArgs& a, const Hit& f) {
  if (!f.on) return 0;
  const uint32_t bit = 1u << (f.e & 31);
  return !(atomicOr(&a.touch[(uint32_t)f.e >> 5], bit) & bit);
}

// Voxel at which the ray S -> q enters world cell c along axis dm (c is not
// the sensor's cell): see the traversal pass below for the tie rule.
//
// At that instant another axis k lies at X_k = (S_k |D| + s_k |D_k| num) / |D|
// (Q units; D = the dominant component, s_k the sign along k, num = the
// dominant-axis distance from the sensor to the cell's boundary), in cell
// floor(X_k / 2^16).  A float estimate of that quotient is within 0.02 of it
// (|S_k| < 2^31, the displacement along k is below 2^27, each float step
// rounds to 2^-24 relative), so its floor is off by at most one and one
// exact 64-bit remainder test each way settles it.  All three axes are
// computed without branches (dm varies across a wave) and the dominant one
// is replaced by c.
__device__ __forceinline__ void entry_voxel(const int32_t S[3], const int32_t sg[3],
                                            const int32_t ad[3], const int dm, const int32_t c,
                                            int32_t v[3]) {
  const int32_t Sd = sel3(dm, S[0], S[1], S[2]);
  const int32_t dd = sel3(dm, ad[0], ad[1], ad[2]);
  const int32_t sd = sel3(dm, sg[0], sg[1], sg[2]);
  // |num| < 2^28 (the ray spans fewer than 2^11 cells); formed from the
  // cell offset so that no intermediate overflows
  const int32_t off = c - (Sd >> 16);
  const int32_t num = sd > 0 ? (off << 16) - (Sd & 0xFFFF) : (Sd & 0xFFFF) - ((off + 1) << 16);
  const int64_t den = (int64_t)dd << 16;
  const float rden = __builtin_amdgcn_rcpf((float)dd * 65536.0f);
  const float fdd = (float)dd, fnum = (float)num;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int32_t sad = sg[k] * ad[k];
    const int64_t x = (int64_t)S[k] * dd + (int64_t)num * sad;
    int64_t qe = (int64_t)floorf(__builtin_fmaf((float)S[k], fdd, fnum * (float)sad) * rden);
    int64_t r = x - ((qe * dd) << 16);
    if (r < 0) {
      qe -= 1;
      r += den;
    } else if (r >= den) {
      qe += 1;
      r -= den;
    }
    if (r == 0 && sd < 0 && sg[k] < 0) qe -= 1;
    v[k] = k == dm ? c : (int32_t)qe;
  }
}

// Exact traversal state of one segment: which axis crosses into its next cell
// first, and the moves left.
//
// Axis k crosses its next cell boundary at time num_k / |D_k| (num = distance
// from the sensor to that boundary along the axis, Q units).  The order of two
// axes is the sign of E_ab = num_a |D_b| - num_b |D_a|, which only changes by
// multiples of 2^16 (|D| << 16 per step): its low 16 bits are fixed, and
// floor(E / 2^16) carries the rest.  When several axes cross at one instant,
// the axes moving up step first, together (the shared boundary belongs to the
// upper cell), the axes moving down in the next step, together.  So a steps
// (before or with b) iff E < 0, or E = 0 and not (a down and b up); b steps iff
// E > 0, or E = 0 and not (a up and b down).  With f = floor(E / 2^16) - d,
// d = 1 when a moves up, b down and the low bits are zero (E = 0 then has to
// read as negative), and g = 1 when both move the same way and the low bits are
// zero: a steps iff f < g, b steps iff f >= 0.
//
// The next boundary of every axis lies within one cell of the current point,
// so |E| <= 2^16 max(|D_a|, |D_b|) < 2^43 and f fits in 32 bits; an axis without
// motion counts as one cell away for ever (num = 2^16).  An axis that has
// reached the end voxel's coordinate needs no check of its own: its next
// crossing comes after the ray's end, at t > 1 (or, moving down with the end on
// a boundary, at t = 1), while an axis with moves left crosses at t < 1 (moving
// up, at t <= 1, which steps first in a tie).
//
// cnt: an axis whose moves to the end voxel reach the move that leaves the
// window or the segment (the walk ends before that voxel) holds the moves
// before that one, and ends the walk by going negative; any other axis holds
// its moves to the end voxel, and they end the walk by all being zero, if no
// axis of the first kind exists (thr: -1 with one, else 0).
struct Walk {
  int32_t fxy, fxz, fyz, gxy, gxz, gyz;
  int32_t ad[3], cnt[3], thr;
};

__device__ __forceinline__ void pair_init(const int32_t num_a, const int32_t ad_a, const bool up_a,
                                          const int32_t num_b, const int32_t ad_b, const bool up_b,
                                          int32_t& f, int32_t& g) {
  const int64_t e = (int64_t)num_a * ad_b - (int64_t)num_b * ad_a;
  const bool exact = (e & 0xFFFF) == 0;
  f = (int32_t)(e >> 16) - (exact & up_a & !up_b);
  g = exact & (up_a == up_b);
}

__device__ __forceinline__ bool walk_ended(const Walk& w) {
  return (w.cnt[0] | w.cnt[1] | w.cnt[2]) <= w.thr;
}

// Starts the walk of a ray to q at world voxel v (inside the window, local l).
// sg, ad: signs and sizes of the ray's displacement.  most[k]: an upper bound
// of the walk's moves along axis k (the dominant axis moves seg_len times at
// most, another one no faster than twice as fast).
__device__ __forceinline__ void walk_init(const InsertArgs& a, const int32_t q[3],
                                          const int32_t v[3], const int32_t l[3],
                                          const int32_t sg[3], const int32_t ad[3], const int dom,
                                          Walk& w, int32_t most[3]) {
  const int32_t dims[3] = {a.d.nx, a.d.ny, a.d.nz};
  int32_t num[3];  // |num| < 2^28: v lies on the ray, which spans fewer than 2^11 cells
  bool stopped = false;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int32_t ev = q[k] >> 16;
    const int32_t rem = ev > v[k] ? ev - v[k] : v[k] - ev;
    int32_t T = (sg[k] > 0 ? dims[k] - 1 - l[k] : l[k]) + 1;  // the move that leaves the window
    T = k == dom ? min(T, a.seg_len) : T;                     // or the segment
    const bool stop = rem >= T;
    stopped |= stop;
    w.cnt[k] = stop ? T - 1 : rem;
    w.ad[k] = ad[k];
    most[k] = min(stop ? T : rem, 2 * a.seg_len + 2);
    const int32_t off = v[k] - (a.S[k] >> 16), fr = a.S[k] & 0xFFFF;
    num[k] = sg[k] > 0 ? ((off + 1) << 16) - fr : fr - (off << 16);
    num[k] = sg[k] == 0 ? 1 << 16 : num[k];
  }
  w.thr = stopped ? -1 : 0;
  pair_init(num[0], ad[0], sg[0] > 0, num[1], ad[1], sg[1] > 0, w.fxy, w.gxy);
  pair_init(num[0], ad[0], sg[0] > 0, num[2], ad[2], sg[2] > 0, w.fxz, w.gxz);
  pair_init(num[1], ad[1], sg[1] > 0, num[2], ad[2], sg[2] > 0, w.fyz, w.gyz);
}

// One step: sets which axes move; the walk has ended when walk_ended() after it.
__device__ __forceinline__ void walk_step(Walk& w, bool& mx, bool& my, bool& mz) {
  mx = (w.fxy < w.gxy) & (w.fxz < w.gxz);
  my = (w.fxy >= 0) & (w.fyz < w.gyz);
  mz = (w.fxz >= 0) & (w.fyz >= 0);
  w.cnt[0] -= mx;
  w.cnt[1] -= my;
  w.cnt[2] -= mz;
  // unsigned adds: a walk that has ended may drift on until its wave's end
  const uint32_t a0 = (uint32_t)w.ad[0], a1 = (uint32_t)w.ad[1], a2 = (uint32_t)w.ad[2];
  w.fxy = (int32_t)((uint32_t)w.fxy + (mx ? a1 : 0u) + (my ? 0u - a0 : 0u));
  w.fxz = (int32_t)((uint32_t)w.fxz + (mx ? a2 : 0u) + (mz ? 0u - a0 : 0u));
  w.fyz = (int32_t)((uint32_t)w.fyz + (my ? a2 : 0u) + (mz ? 0u - a1 : 0u));
}

// a * b + c on the 24-bit multiplier (operands below 2^24; b uniform across
// the wave, taken from a scalar register).  Written out because the compiler
// widens the plain expression into a 64-bit multiply-add when the result
// feeds an address.
__device__ __forceinline__ uint32_t mad_u24(uint32_t a, uint32_t b, uint32_t c) {
  uint32_t r;
  asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
  return r;
}

// Storage index of voxel (sx, sy, sz) from sx, 4 sy and 16 sz, with 24-bit
// multiplies: brick coordinates < 2^11, nby <= 2048 and 16 nz <= 2048 keep every
// operand within 24 bits, and the index is below 2^31 for every map the library
// accepts.
__device__ __forceinline__ int32_t index24(const Dims& d, int32_t sx, int32_t sy4, int32_t sz16) {
  const uint32_t b = mad_u24((uint32_t)(sx >> 2), (uint32_t)d.nby, (uint32_t)(sy4 >> 4));
  const uint32_t low = (((uint32_t)sx & 3u) | ((uint32_t)sy4 & 12u)) | (uint32_t)sz16;
  return (int32_t)mad_u24(b, (uint32_t)d.nz << 4, low);
}

}  // namespace
}  // namespace gvom
