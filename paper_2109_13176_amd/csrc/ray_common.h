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
// so |E| <= 2^16 max(|D_a|, |D_b|) < 2^43 and f fits in 32 bits; against an axis
// without motion (taken as moving up: its boundary lies ahead) E never changes and
// has the sign that lets the other one step.  An axis that has
// reached the end voxel's coordinate needs no check of its own: its next
// crossing comes after the ray's end, at t > 1 (or, moving down with the end on
// a boundary, at t = 1), while an axis with moves left crosses at t < 1 (moving
// up, at t <= 1, which steps first in a tie).
//
// pos holds cnt << 16 | storage coordinate, so that one addition counts a move and
// makes it.  cnt: an axis whose moves to the end voxel reach the move that leaves the
// window or the segment (the walk ends before that voxel) holds the moves
// before that one, and ends the walk by going negative; any other axis holds
// its moves to the end voxel, and they end the walk by all being zero, if no
// axis of the first kind exists (thr: -1 with one, else 2^16 - 1).
struct Walk {
  int32_t fxy, fxz, fyz, gxy, gxz, gyz;
  int32_t ad[3], na[2], thr;  // |D|, -|D_x| and -|D_y|
  int32_t pos[3];   // cnt << 16 | storage coordinate (sx, 4 sy, 16 sz)
  int32_t move[3];  // what a move adds to pos
};

__device__ __forceinline__ bool walk_ended(const Walk& w) {
  return (w.pos[0] | w.pos[1] | w.pos[2]) <= w.thr;
}

// Starts the walk of segment j of the ray to q with dominant axis dom (j the same
// for the whole wave): l = local coordinates of its first voxel; up[k]: the ray
// does not move down along axis k; most[k]: an upper bound of the walk's moves
// along axis k: those left to the end voxel and one past it, or, where the segment is
// shorter, those of a segment.  The dominant axis d, which has the most voxel steps n_d,
// moves seg_len times in it; another axis k moves at |D_k| / |D_d| < (n_k + 1) / (n_d - 1)
// times its speed.  For n_d >= 3 that is at most 2: 2 seg_len + 2 moves.  For n_d <= 2 it
// may be any number, but then the first bound is at most 3 moves, and the other one 4.
// False when the first voxel lies outside the window.
//
// Along axis k the ray reaches its (i + 1)-st boundary after h_k + 2^16 i Q units,
// h_k the distance from the sensor to the first one.  Segment j > 0 starts when the
// dominant axis (d) has moved num = h_d + 2^16 (J - 1), J = j seg_len, and has made
// J moves; another axis k has then made the moves m whose boundaries it has
// reached, h_k |D_d| + 2^16 (m - 1) |D_d| <= num |D_k| (< when it moves down and d up:
// a shared boundary belongs to the upper cell).  That is the quotient of
// y = num |D_k| + (2^16 - h_k) |D_d| by 2^16 |D_d|, and the remainder r of that
// division is what the walk starts from: E_dk = r + 2^16 (|D_k| - |D_d|).  (With j = 0
// the same holds for m = 0 and r = y, which then is no remainder.)
//
// The quotient is below 2^12; its float estimate is within 0.01 of it, so lowered
// by 0.02 and truncated it is the quotient or one less, which one exact comparison of
// the remainder settles.  For < instead of <=, the same is done with y - 1.
//
// Axes in the order d, b, c (the others in ascending order), only at the end
// brought back to x, y, z: the quotients are taken for two axes instead of three,
// and two of the three E need no product of their own.  (Three entry coordinates and
// three E, each by its own products: 390 vector instructions in the code and 27 wide
// multiplies, so 270 and 12.)
__device__ __forceinline__ bool segment_init(const InsertArgs& a, const int32_t q[3], const int dom,
                                             const int32_t j, Walk& w, int32_t l[3], bool up[3],
                                             int32_t most[3]) {
  const int32_t dims[3] = {a.d.nx, a.d.ny, a.d.nz};
  const int32_t J = j * a.seg_len;
  // (numbers that are never negative as unsigned: their products take one
  // multiply-add; truth values as 0 / 1)
  uint32_t ad[3], h[3], u[3];
  int32_t n[3];
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int32_t dq = q[k] - a.S[k], dv = (q[k] >> 16) - (a.S[k] >> 16), fr = a.S[k] & 0xFFFF;
    up[k] = dq >= 0;
    u[k] = up[k];
    ad[k] = (uint32_t)(up[k] ? dq : -dq);
    w.ad[k] = (int32_t)ad[k];
    n[k] = up[k] ? dv : -dv;
    h[k] = (uint32_t)(up[k] ? 65536 - fr : fr);
  }
  const bool d0 = dom == 0, d1 = dom == 1, d2 = dom == 2;
  const uint32_t dd = d0 ? ad[0] : d1 ? ad[1] : ad[2], hd = d0 ? h[0] : d1 ? h[1] : h[2];
  const uint32_t adk[2] = {d0 ? ad[1] : ad[0], d2 ? ad[1] : ad[2]};
  const uint32_t hk[2] = {d0 ? h[1] : h[0], d2 ? h[1] : h[2]};
  uint32_t m[2] = {0, 0}, xd[2];  // xd: E_dk is a multiple of 2^16
  int32_t fd[2];
  if (j > 0) {
    const uint32_t ud = d0 ? u[0] : d1 ? u[1] : u[2];
    const uint32_t uk[2] = {d0 ? u[1] : u[0], d2 ? u[1] : u[2]};
    const uint32_t num = hd + ((uint32_t)(J - 1) << 16);
    const float fdd = (float)dd, fnum = (float)num;
    const float rden = __builtin_amdgcn_rcpf(fdd * 65536.0f);
    const uint64_t den = (uint64_t)dd << 16;
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const uint32_t g = 65536 - hk[k], strict = ud & ~uk[k];
      const float est = __builtin_fmaf(fnum, (float)adk[k], (float)g * fdd) * rden;
      m[k] = (uint32_t)(int32_t)(est - 0.02f);
      uint64_t r = (uint64_t)num * adk[k] + (uint64_t)g * dd - strict - (uint64_t)(m[k] << 16) * dd;
      const bool more = r >= den;
      m[k] += more;
      r = r - (more ? den : 0) + strict;
      xd[k] = ((uint32_t)r & 0xFFFF) == 0;
      fd[k] = (int32_t)((uint32_t)(r >> 16) + adk[k] - dd);
    }
  } else {
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const uint64_t e = (uint64_t)hd * adk[k] - (uint64_t)hk[k] * dd;
      xd[k] = ((uint32_t)e & 0xFFFF) == 0;
      fd[k] = (int32_t)(e >> 16);
    }
  }
  const uint64_t e = (uint64_t)(hk[0] + (m[0] << 16)) * adk[1] - (uint64_t)(hk[1] + (m[1] << 16)) * adk[0];
  const int32_t fbc = (int32_t)(e >> 16);
  const uint32_t xbc = ((uint32_t)e & 0xFFFF) == 0;
  // floor(-E / 2^16)
  const int32_t nb = ~fd[0] + (int32_t)xd[0], nc = ~fd[1] + (int32_t)xd[1];
  const uint32_t xxy = d2 ? xbc : xd[0], xxz = d0 ? xd[1] : d1 ? xbc : xd[0], xyz = d0 ? xbc : xd[1];
  w.fxy = (d0 ? fd[0] : d1 ? nb : fbc) - (int32_t)(xxy & u[0] & ~u[1]);
  w.fxz = (d0 ? fd[1] : d1 ? fbc : nb) - (int32_t)(xxz & u[0] & ~u[2]);
  w.fyz = (d0 ? fbc : d1 ? fd[1] : nc) - (int32_t)(xyz & u[1] & ~u[2]);
  w.gxy = (int32_t)(xxy & ~(u[0] ^ u[1]));
  w.gxz = (int32_t)(xxz & ~(u[0] ^ u[2]));
  w.gyz = (int32_t)(xyz & ~(u[1] ^ u[2]));
  const int32_t mv[3] = {d0 ? J : (int32_t)m[0], (int32_t)(d0 ? m[0] : d1 ? (uint32_t)J : m[1]),
                         d2 ? J : (int32_t)m[1]};
  bool inside = true, stopped = false;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const int32_t ls = (a.S[k] >> 16) - a.O[k];
    l[k] = ls + (up[k] ? mv[k] : -mv[k]);
    inside &= (uint32_t)l[k] < (uint32_t)dims[k];
    // moves from the sensor's voxel to the one that leaves the window or the segment
    int32_t T = up[k] ? dims[k] - ls : ls + 1;
    T = k == dom ? min(T, J + a.seg_len) : T;
    stopped |= n[k] >= T;
    const int32_t cnt = min(n[k], T - 1) - mv[k];
    w.pos[k] = (int32_t)((uint32_t)cnt << 16);
    w.move[k] = -(1 << 16);
    most[k] = min(cnt + 1, 2 * a.seg_len + 2);
  }
  w.thr = stopped ? -1 : 0xFFFF;
  w.na[0] = -w.ad[0];
  w.na[1] = -w.ad[1];
  asm("" : "+v"(w.na[0]), "+v"(w.na[1]));  // kept: a sum of three, not a difference and a sum
  return inside;
}

// One step; the walk has ended when walk_ended() after it.
__device__ __forceinline__ void walk_step(Walk& w) {
  const bool mx = (w.fxy < w.gxy) & (w.fxz < w.gxz);
  const bool my = (w.fxy >= 0) & (w.fyz < w.gyz);
  const bool mz = (w.fxz >= 0) & (w.fyz >= 0);
  w.pos[0] += mx ? w.move[0] : 0;
  w.pos[1] += my ? w.move[1] : 0;
  w.pos[2] += mz ? w.move[2] : 0;
  w.fxy = w.fxy + (mx ? w.ad[1] : 0) + (my ? w.na[0] : 0);
  w.fxz = w.fxz + (mx ? w.ad[2] : 0) + (mz ? w.na[0] : 0);
  w.fyz = w.fyz + (my ? w.ad[2] : 0) + (mz ? w.na[1] : 0);
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

// Storage index of the voxel at pos (Walk::pos), with 24-bit multiplies: brick
// coordinates < 2^11, nby <= 2048 and 16 nz <= 2048 keep every operand within 24
// bits, and the index is below 2^31 for every map the library accepts.
__device__ __forceinline__ int32_t index24(const Dims& d, const int32_t pos[3]) {
  const uint32_t x = (uint32_t)pos[0], y = (uint32_t)pos[1], z = (uint32_t)pos[2] & 0xFFFFu;
  const uint32_t b = mad_u24((x >> 2) & 0x3FFFu, (uint32_t)d.nby, (y >> 4) & 0xFFFu);
  uint32_t low;  // x's two low bits, y's others; the compiler finds no bit select in it
  asm("v_bfi_b32 %0, 3, %1, %2" : "=v"(low) : "v"(x), "v"(y));
  low = (low & 15u) | z;
  return (int32_t)mad_u24(b, (uint32_t)d.nz << 4, low);
}

__device__ __forceinline__ int32_t pos_x(const Walk& w) { return w.pos[0] & 0xFFFF; }
__device__ __forceinline__ int32_t pos_y(const Walk& w) { return (w.pos[1] >> 2) & 0x3FFF; }
__device__ __forceinline__ int32_t pos_z(const Walk& w) { return (w.pos[2] >> 4) & 0xFFF; }

// Brings a coordinate along axis k that a move took past either end of the
// storage (n voxels; read as an unsigned number -1 lies past the end too) to the
// other end.
__device__ __forceinline__ void wrap_pos(Walk& w, const int k, const int32_t n) {
  const int32_t size = n << (2 * k);
  const bool out = (w.pos[k] & 0xFFFF) >= size;
  const int32_t by = (int16_t)w.move[k] < 0 ? size : -size;
  w.pos[k] += out ? by : 0;
}

}  // namespace
}  // namespace gvom
