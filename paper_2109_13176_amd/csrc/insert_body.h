// Device bodies of the scan-insertion kernels (Sec. III-C of arXiv 2109.13176):
// the ray pass, the traversal with its line tables and sensor box, the
// sensor-box fold and the window-scroll clears.  Each body does the work of
// one (virtual) block, so the single-map kernels and the batched persistent
// kernel share them.
#pragma once
#include <math.h>

#include <type_traits>

#include "ray_common.h"

namespace gvom {

namespace {


// ---------------------------------------------------------------------------
// Pass 1, one lane per point: transform, and cut the ray into segments for the
// traversal pass.  It touches nothing of the map, so the clears of the moved
// window run beside it (in a launch of their own before it they took 3-6 us, on
// 1024 x 1024 x 96 34 us); the traversal pass records the returns.  With the
// clears: 5.8 + 8.2 -> 7.1 us for 131,072 points on 512 x 512 x 64.
//
// A ray's voxel path is monotone in every axis.  Along its dominant axis (the
// axis with the most voxel steps) the path is cut every seg_len voxels:
// segment j holds the path voxels whose dominant coordinate lies j*seg_len ..
// (j+1)*seg_len - 1 voxels from the sensor's.  Only segments that start
// inside the window along the dominant axis count.
//
// The block then regroups its rays by segment count (most first; rays of
// equal count keep their order, so neighbouring rays stay together) and
// writes their records {Q, 4 segments + dominant axis} in that order: a traversal wave holds
// segment j of 64 rays that all have it, instead of 64 neighbouring rays of
// which the short ones ended long before j.  Each group of 64 records with at
// most s segments publishes s wave items {group, j}.
constexpr int kRayWaves = kRayBlock / 64;
constexpr int kSegBins = 64;  // segment counts >= kSegBins - 1 share a bin
static_assert(kSegBins * kRayWaves == kRayBlock, "one scan entry per thread");

// Exclusive prefix sum over the block (one value per thread); wtot is
// kRayWaves words of the caller's LDS.
__device__ __forceinline__ int block_excl_scan(int v, int* wtot) {
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(x, o);
    if (lane >= o) x += y;
  }
  if (lane == 63) wtot[wv] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int s = 0;
    for (int w = 0; w < kRayWaves; w++) {
      const int c = wtot[w];
      wtot[w] = s;
      s += c;
    }
  }
  __syncthreads();
  return x - v + wtot[wv];
}

// First wave item of stripe t: the ray blocks t, t + kStripes, ... of the stripes
// before it have room for block_items each.
__device__ __forceinline__ int64_t stripe_off(const InsertArgs& a, const int t) {
  const uint32_t blocks = ((uint32_t)a.n + kRayBlock - 1) / kRayBlock;
  const uint32_t some = blocks % kStripes;
  return (int64_t)a.block_items * ((uint32_t)t * (blocks / kStripes) + ((uint32_t)t < some ? t : some));
}

__device__ __forceinline__ void rays_body(const InsertArgs& a, const int blk) {
  __shared__ unsigned int wcount[kRayWaves][4];
  __shared__ unsigned long long wbase[kRayWaves];
  __shared__ int bin_pre[kSegBins * kRayWaves];  // [bin][wave]: count, then prefix
  __shared__ int wtot[kRayWaves];
  __shared__ int4 srec[kRayBlock];
  const int lane = __lane_id(), wv = threadIdx.x >> 6;
  const int i = blk * kRayBlock + threadIdx.x;
  const int32_t dims[3] = {a.d.nx, a.d.ny, a.d.nz};
  int32_t q[3];
  PointFlags pf;
  const bool ray = point_pass(a, i, q, pf);
  const bool nonfinite = pf.nonfinite, outrange = pf.outrange, hit = pf.hit;

  int nseg = 0;  // of a ray at least 1 (one that ends in the sensor's voxel has no steps)
  int axis = 0;  // its dominant axis
  if (ray) {
    int32_t n[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const int32_t sv = a.S[k] >> 16, ev = q[k] >> 16;
      n[k] = ev > sv ? ev - sv : sv - ev;
    }
    const int dom = dominant_axis(n);
    const int32_t Sd = sel3(dom, a.S[0], a.S[1], a.S[2]);
    const int32_t lc = (Sd >> 16) - sel3(dom, a.O[0], a.O[1], a.O[2]);
    const int32_t room = sel3(dom, q[0], q[1], q[2]) > Sd ? sel3(dom, dims[0], dims[1], dims[2]) - 1 - lc : lc;
    nseg = min(sel3(dom, n[0], n[1], n[2]), room) / a.seg_len + 1;
    axis = dom;
  }

  // ---- stable counting sort of the block's rays by bin (most segments first)
  const int bin = kSegBins - 1 - min(nseg, kSegBins - 1);
  unsigned long long peers = ~0ull;  // lanes of this wave in the same bin
#pragma unroll
  for (int k = 0; k < 6; k++) {
    const bool bit = (bin >> k) & 1;
    const unsigned long long m = __ballot(bit);
    peers &= bit ? m : ~m;
  }
  const int rank = __popcll(peers & ((1ull << lane) - 1ull));
  bin_pre[threadIdx.x] = 0;
  __syncthreads();
  if (rank == 0) bin_pre[bin * kRayWaves + wv] = __popcll(peers);
  __syncthreads();
  const int pre = block_excl_scan(bin_pre[threadIdx.x], wtot);
  bin_pre[threadIdx.x] = pre;  // every thread read its entry before the scan's barriers
  __syncthreads();
  srec[bin_pre[bin * kRayWaves + wv] + rank] = make_int4(q[0], q[1], q[2], nseg << 2 | axis);
  __syncthreads();
  const int4 rec = srec[threadIdx.x];
  a.rays[i] = rec;

  // ---- reserve the wave items: one returning atomic per block, group bases
  // from the block's prefix
  int maxseg = rec.w >> 2;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) maxseg = max(maxseg, __shfl_xor(maxseg, o));
  const int c0 = __popcll(__ballot(nonfinite));
  const int c1 = __popcll(__ballot(outrange));
  const int c2 = __popcll(__ballot(hit));
  if (lane == 0) {
    wcount[wv][0] = maxseg;
    wcount[wv][1] = c0;
    wcount[wv][2] = c1;
    wcount[wv][3] = c2;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long sum = 0, s0 = 0, s1 = 0, s2 = 0;
    for (int w = 0; w < kRayWaves; w++) {
      wbase[w] = sum;
      sum += wcount[w][0];
      s0 += wcount[w][1];
      s1 += wcount[w][2];
      s2 += wcount[w][3];
    }
    // blocks are spread over kStripes counters, each with its own item region
    const int st = blk % kStripes;
    const unsigned long long b = sum ? atomicAdd(&a.stats[8 + st], sum) : 0ull;
    for (int w = 0; w < kRayWaves; w++) wbase[w] += b + stripe_off(a, st);
    unsigned long long* pr = a.part_rays + 4 * (size_t)blk;
    pr[0] = s0;
    pr[1] = s1;
    pr[2] = s2;
    pr[3] = 0;
  }
  __syncthreads();
  const int gw = blk * kRayWaves + wv;  // this group's rays: 64 gw .. 64 gw + 63
  const unsigned long long off = wbase[wv];
  for (int j = lane; j < maxseg; j += 64) a.witems[off + j] = make_int2(gw, j);
}

// ---------------------------------------------------------------------------
// Inclusive prefix sums over the first kStripes = 16 lanes (one DPP row).
__device__ __forceinline__ int64_t stripe_scan(int64_t v) {
  const auto add = [&](auto c) {
    constexpr int kRowShr = decltype(c)::value;
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)v, kRowShr, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), kRowShr, 0xf, 0xf, true);
    v += (int64_t)((uint64_t)hi << 32 | lo);
  };
  add(std::integral_constant<int, 0x111>());
  add(std::integral_constant<int, 0x112>());
  add(std::integral_constant<int, 0x114>());
  add(std::integral_constant<int, 0x118>());
  return v;
}

__device__ __forceinline__ int64_t read_lane64(const int64_t v, const int lane) {
  const uint32_t lo = __builtin_amdgcn_readlane((int)v, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((int)(v >> 32), lane);
  return (int64_t)((uint64_t)hi << 32 | lo);
}

// Pass 2: record the returns, one lane per ray, then, one lane per ray segment,
// walk the segment voxel by voxel and add one pass to every window voxel before
// the ray's end voxel.  (The returns' reads and atomics overlap the set-up of
// the blocks' tables and the stripe counts' round trip.)
//
// Start voxel of segment j > 0: the instant the dominant axis enters cell
// c = c_sensor +- j*seg_len, at exact time t = num / |D_dom|.  Another axis b
// then lies in cell floor(X_b(t)); if X_b(t) is exactly on a boundary while
// both b and the dominant axis move down, b leaves its cell at the same
// instant as the dominant axis (one cell lower).
//
// Traversal: along axis a the segment leaves its current cell when it has
// moved num_a (Q units) at speed |D_a|, i.e. at time num_a / |D_a|.  The axis
// with the smallest time steps next; times are compared exactly through the
// pairwise differences E_ab = num_a |D_b| - num_b |D_a|, which change by
// constant increments when an axis steps (kept as 32-bit high parts, see
// Walk).  When several axes share the smallest time, the axes moving up step
// first (the shared boundary belongs to the upper cell) and the axes moving
// down step in the next iteration, so the voxel at that instant is visited.
//
// Counting.  Device atomics are charged per (instruction, 64-byte line) at
// the memory side, and the 64 rays of a wave item pass a compact set of lines
// (about 15 on the 64-beam workload, against about 60 line requests when
// every step adds its voxels straight to the map).  So each wave counts its
// item in a private LDS line table: kWtSlots slots of one 64-byte storage
// line each (16 counters of 8 bits, four per word: a voxel takes at most one
// pass per lane of the item, so a counter stays below 65 while it is in the
// table; and a tag = storage index >> 4), found by a hash of
// the line with up to kWtProbe more probes and claimed by compare-and-swap.  A step
// reads one tag, that of its lane's slot or, on another line, of the line's home
// slot, and moves to the next voxel before it looks at it; only lanes that find
// another line there search.  When the item is done the wave adds every non-zero
// counter of its claimed slots to the map, 16 lanes per line (one line request
// per line), and empties the table.  A line that finds no slot on its probe
// path is added to the map directly.  With BOX, voxels in the sensor box add
// into the block's LDS copy of the box instead, which the block flushes into
// its replica at the end (k_box_fold adds the replicas into the map).  Every
// pass ends up in exactly one counter that reaches the map once, so the
// result is the same integer sum whatever the claim order.
//
// On 512 x 512 x 64 with 131,072 points the walk makes 150,000 wave steps (three lanes of
// four active) in 16,800 items of segments of 5 voxels, or 146,000 in 10,700 of 8: 17.9 M
// and 16.0 M vector instructions in all.  Their issue fills two thirds of the kernel's
// time; on 128 x 128 x 32 with 28,800 points, with one wave per SIMD, the chain of LDS
// and memory round trips does.  With 16-bit counters, a search at every change of line,
// coordinates, wraps and move counts in registers of their own, the stripes searched in
// LDS and a set-up by divisions: 46.4 and 19.8 us, then 43.1 and 16.0 (segments of 8).
constexpr int kWtSlots = 64;     // slots per wave (one per lane at the flush)
constexpr int kWtStride = 5;     // LDS words per slot: tag and 4 words of 4 counters
constexpr int kWtProbe = 4;
constexpr int32_t kWtEmpty = -1;


struct WaveTable {
  uint32_t slot[(kWtSlots + 1) * kWtStride];  // {tag, 4 words of counters}; the last: see wt_claim
  int32_t lst[kWtSlots];
};

// Orders the LDS accesses of one wave's lanes (a wave's LDS operations are
// executed in issue order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Byte offset in the block's tables (this wave's begins at `base`) of the slot where the search for storage line
// `line` begins: a multiplicative (Fibonacci) hash of the line's low 24 bits, the
// top six bits of their product with 2^24 / golden ratio (Knuth, TAOCP vol. 3,
// 6.4), one 24-bit multiply.  Tags hold the whole line, so lines that share
// low bits only share a probe path.
__device__ __forceinline__ uint32_t wt_home(const int32_t line, const uint32_t base) {
  const uint32_t h = (uint32_t)__umul24((uint32_t)line, 0x9E3779u) >> 26;
  return (uint32_t)__umul24(h, 4 * kWtStride) + base;
}

__device__ __forceinline__ uint32_t* wt_word(WaveTable* wtab, const uint32_t at) {
  return (uint32_t*)((char*)wtab + at);
}

constexpr uint32_t kWtLast = 4 * kWtStride * (kWtSlots - 1);  // offset of the last slot

// The slot of `line` whose home slot `at` holds the tag t, not that line: claims
// an empty slot or finds the line's on the rest of its probe path, one
// compare-and-swap per probe.  When the path holds other lines only, the slot
// behind the table, which nothing reads and no line is found in.
__device__ __forceinline__ uint32_t wt_claim(WaveTable* wtab, const uint32_t base,
                                             const int32_t line, uint32_t at, const int32_t t) {
  const auto next = [&](uint32_t x) { return x == base + kWtLast ? base : x + 4u * kWtStride; };
  if (t != kWtEmpty) at = next(at);
  for (int p = 0;;) {
    const int32_t o = (int32_t)atomicCAS(wt_word(wtab, at), (uint32_t)kWtEmpty, (uint32_t)line);
    if (o == kWtEmpty || o == line) return at;
    if (++p == kWtProbe) return base + kWtLast + 4u * kWtStride;
    at = next(at);
  }
}

// box_cnt[kBoxCells] and wtab[NT / 64] are the block's LDS (the caller's).
template <bool DISTINCT, bool BOX, int NT>
__device__ __forceinline__ void trace_body(const InsertArgs& a, const int blk, const int nblk,
                                           int32_t* box_cnt, WaveTable* wtab) {
  const int lane = __lane_id();
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  WaveTable& wt = wtab[wave];
  const uint32_t base = (uint32_t)(wave * sizeof(WaveTable));
  const int64_t slots = ((int64_t)a.n + kRayBlock - 1) / kRayBlock * kRayBlock;  // ray records
  const int slot0 = blk * NT + (int)threadIdx.x;
  int4 ray0 = make_int4(0, 0, 0, 0);
  unsigned long long cnt0 = 0;  // items of stripe `lane`
  if (lane < kStripes) cnt0 = a.stats[8 + lane];
  if (slot0 < slots) ray0 = a.rays[slot0];
  for (int i = lane; i < kWtSlots * kWtStride; i += 64) wt.slot[i] = 0;
  wave_lds_sync();
  wt.slot[lane * kWtStride] = (uint32_t)kWtEmpty;
  if (BOX) {
    for (int i = threadIdx.x; i < kBoxCells; i += NT) box_cnt[i] = 0;
  }
  const int nx = a.d.nx, ny = a.d.ny, nz = a.d.nz;
  const int32_t dims[3] = {nx, ny, nz};
  // Wave items of stripe t: [stripe_off(t), stripe_off(t) + count), item u of all
  // belongs to the last stripe whose prefix is <= u (empty stripes share their
  // prefix).  Lane t < kStripes holds stripe t's prefix, and what takes u to its
  // place in a.witems.
  const int64_t stride = (int64_t)nblk * (NT / 64);
  int64_t u = (int64_t)blk * (NT / 64) + wave;
  const int64_t off = stripe_off(a, lane);
  const int64_t mine = lane < kStripes ? min((int64_t)cnt0, stripe_off(a, lane + 1) - off) : 0;
  const int64_t incl = stripe_scan(mine);
  const int64_t pre = incl - mine, to_item = off - pre;
  const int64_t count = read_lane64(incl, kStripes - 1);  // wave items
  const auto find_item = [&](int64_t x) {
    const int t = __popcll(__builtin_amdgcn_ballot_w64(lane < kStripes && x >= pre)) - 1;
    return a.witems[read_lane64(to_item, t) + x];
  };
  int2 item = make_int2(0, 0);
  if (u < count) item = find_item(u);
  const Hit hit0 = find_hit(a, ray0);
  const HitReads reads0 = record_hit_issue(a, hit0);
  uint32_t* touch_p = DISTINCT ? a.touch + ((a.d.vs + 31) >> 5) : nullptr;
  int32_t* const passes = a.passes;  // kept in registers across the loop
  int n_pass = 0, n_dpass = 0, n_upd = 0;
  int n_dhit = 0;
  record_hit_finish(a, hit0, reads0, ray0.z);
  if (DISTINCT) n_dhit += distinct_hit(a, hit0);
  for (int64_t i = (int64_t)slot0 + (int64_t)nblk * NT; i < slots; i += (int64_t)nblk * NT) {
    const int4 r = a.rays[i];
    const Hit h = find_hit(a, r);
    record_hit_finish(a, h, record_hit_issue(a, h), r.z);
    if (DISTINCT) n_dhit += distinct_hit(a, h);
  }
  if (BOX) __syncthreads();  // the box is zero

  bool touched = false;
  for (; u < count; u += stride) {
    const int j = __builtin_amdgcn_readfirstlane(item.y);
    const int4 ray = a.rays[(int64_t)__builtin_amdgcn_readfirstlane(item.x) * 64 + lane];
    bool active = false, wrap[3] = {false, false, false};
    Walk w = {};
    int32_t sidx = 0;
    {
      const int32_t q[3] = {ray.x, ray.y, ray.z};
      int32_t l[3], most[3];
      bool up[3];
      const bool inside = segment_init(a, q, ray.w & 3, j, w, l, up, most);
      active = inside && j < ray.w >> 2 && !walk_ended(w);  // (j: the ray has segment j)
#pragma unroll
      for (int k = 0; k < 3; k++) {
        const int32_t s = wrap_add(l[k] + a.d.ro[k], dims[k]);
        wrap[k] = active && (up[k] ? s + most[k] >= dims[k] : s < most[k]);
        w.pos[k] += s << (2 * k);
        w.move[k] += up[k] ? 1 << (2 * k) : -(1 << (2 * k));
      }
      sidx = index24(a.d, w.pos);
    }
    // the storage wrap only along axes where a walk of the wave can reach it
    bool wrap_any[3];
#pragma unroll
    for (int k = 0; k < 3; k++) wrap_any[k] = __builtin_amdgcn_ballot_w64(wrap[k]) != 0;
    // box lookups only in waves that can reach the box
    const bool wnear = BOX && j * a.seg_len <= a.box_far;
    touched |= wnear;
    int32_t cur_line = kWtEmpty;  // this lane's current line and its slot
    uint32_t cur_at = 0;
    const auto walk = [&](auto near_c) {
      constexpr bool NEAR = decltype(near_c)::value;
      do {
        n_pass++;
        // ---- the current voxel's slot (read while the step is computed)
        const int32_t line = (int32_t)((uint32_t)sidx >> 4);
        const uint32_t home = wt_home(line, base);
        uint32_t at = line == cur_line ? cur_at : home;
        const int32_t tag = (int32_t)*wt_word(wtab, at);
        const int32_t idx = sidx;
        int bidx = -1;
        if (NEAR) {
          // storage offsets from the box's first cell (unsigned: wrapped)
          const uint32_t d0 = (uint32_t)wrap_add(pos_x(w) - a.box_s[0] + nx, nx);
          const uint32_t d1 = (uint32_t)wrap_add(pos_y(w) - a.box_s[1] + ny, ny);
          const uint32_t d2 = (uint32_t)wrap_add(pos_z(w) - a.box_s[2] + nz, nz);
          if (d0 < (uint32_t)a.box_e[0] && d1 < (uint32_t)a.box_e[1] && d2 < (uint32_t)a.box_e[2])
            bidx = (int)((d0 * kBoxXY + d1) * kBoxZ + d2);
        }
        // ---- step
        walk_step(w);
        if (wrap_any[0]) wrap_pos(w, 0, nx);
        if (wrap_any[1]) wrap_pos(w, 1, ny);
        if (wrap_any[2]) wrap_pos(w, 2, nz);
        sidx = index24(a.d, w.pos);
        // ---- one pass of the voxel
        if (NEAR && bidx >= 0) {
          atomicAdd(&box_cnt[bidx], 1);
        } else {
          cur_line = line;
          if (tag != line) {
            at = wt_claim(wtab, base, line, at, tag);
            if (at == base + kWtLast + 4u * kWtStride) {
              cur_line = kWtEmpty;
              n_upd++;
              atomicAdd(&passes[idx], 1);
              if (DISTINCT) {
                const uint32_t bit = 1u << (idx & 31);
                const uint32_t old = atomicOr(&touch_p[(uint32_t)idx >> 5], bit);
                n_dpass += !(old & bit);
              }
            }
          }
          cur_at = at;
          // counter idx & 15 = byte idx & 3 of word (idx & 15) / 4 (a shift takes 5 bits)
          atomicAdd(wt_word(wtab, at + 4 + (idx & 12)), 1u << ((idx << 3) & 31));
        }
      } while (!walk_ended(w));
    };
    if (active) {
      if (wnear)
        walk(std::true_type());
      else
        walk(std::false_type());
    }
    if (u + stride < count) item = find_item(u + stride);
    // ---- flush the wave's table: 16 lanes per claimed line
    wave_lds_sync();
    const int32_t tg = (int32_t)wt.slot[lane * kWtStride];
    const unsigned long long vm = __builtin_amdgcn_ballot_w64(tg != kWtEmpty);
    if (vm) {
      if (tg != kWtEmpty) wt.lst[__popcll(vm & ((1ull << lane) - 1ull))] = lane * kWtStride;
      wave_lds_sync();
      const int nv = __popcll(vm);
      const int w = lane & 15;
      for (int k = 0; k < nv; k += 4) {
        const int e = k + (lane >> 4);
        if (e < nv) {
          const int s = wt.lst[e];
          const uint32_t four = wt.slot[s + 1 + (w >> 2)];
          const int c = (int)((four >> (8 * (w & 3))) & 0xFFu);
          // the four lanes of a word have read it before the first clears it
          if (four && !(w & 3)) wt.slot[s + 1 + (w >> 2)] = 0;
          if (c) {
            const int32_t addr = ((int32_t)wt.slot[s] << 4) + w;
            n_upd++;
            atomicAdd(&passes[addr], c);
            if (DISTINCT) {
              const uint32_t bit = 1u << (addr & 31);
              const uint32_t old = atomicOr(&touch_p[(uint32_t)addr >> 5], bit);
              n_dpass += !(old & bit);
            }
          }
        }
      }
      wave_lds_sync();
      wt.slot[lane * kWtStride] = (uint32_t)kWtEmpty;
      wave_lds_sync();
    }
  }
  if (BOX) {
    // flush the block's box counts into its replica (coalesced; zero cells
    // are skipped, and blocks none of whose items came near)
    int32_t* rep = a.box_rep + (size_t)(blk % kBoxReps) * kBoxCells;
    const bool any = __syncthreads_or(touched);
    for (int i = any ? (int)threadIdx.x : kBoxCells; i < kBoxCells; i += NT) {
      const int32_t c = box_cnt[i];
      if (c) atomicAdd(&rep[i], c);
    }
  }
  // per-block counters, written without atomics (summed by the host)
  __shared__ int wsum[NT / 64][4];
  const int c3 = wave_sum(n_pass);
  const int c5 = DISTINCT ? wave_sum(n_dhit) : 0;
  const int c4 = DISTINCT ? wave_sum(n_dpass) : 0;
  const int c6 = wave_sum(n_upd);
  if (lane == 0) {
    wsum[threadIdx.x >> 6][0] = c3;
    wsum[threadIdx.x >> 6][1] = c4;
    wsum[threadIdx.x >> 6][2] = c6;
    wsum[threadIdx.x >> 6][3] = c5;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long p = 0, q = 0, u = 0, h = 0;
    for (int w = 0; w < NT / 64; w++) {
      p += wsum[w][0];
      q += wsum[w][1];
      u += wsum[w][2];
      h += wsum[w][3];
    }
    a.part_trace[4 * blk] = p;
    a.part_trace[4 * blk + 1] = q;
    a.part_trace[4 * blk + 2] = u;
    a.part_trace[4 * blk + 3] = h;
  }
}

// Sensor-box fold: thread (cell i, group g) sums cell i over the kFoldReps
// replicas of group g (zeroing them for the next insert) and adds the sum to
// the cell's passes.  Distinct passes of box cells are counted here (the
// traversal skipped them): the group whose bit-or finds the cell's bit clear
// counts it.  Block b (linear over the grid) writes its counters to slot
// trace_blocks + b.
constexpr int kFoldReps = 8;
constexpr int kFoldGroups = kBoxReps / kFoldReps;
static_assert(kBoxReps % kFoldReps == 0, "replica groups");

constexpr int kFoldCellBlocks = (kBoxCells + kBlock - 1) / kBlock;

// Fold block (cell block bx, replica group by) of one map.  Block (0, 0)
// also zeroes the ray pass's segment counters for the next insert (the
// traversal, which read them, has finished).
template <bool DISTINCT>
__device__ __forceinline__ void box_fold_body(const InsertArgs& a, const int bx, const int by) {
  if (bx == 0 && by == 0 && threadIdx.x < kStripes) a.stats[8 + threadIdx.x] = 0ull;
  const int i = bx * kBlock + threadIdx.x;
  int n_dpass = 0;
  if (i < kBoxCells) {
    int32_t v[kFoldReps];
    int32_t* p = a.box_rep + (size_t)by * kFoldReps * kBoxCells + i;
#pragma unroll
    for (int r = 0; r < kFoldReps; r++) v[r] = p[(size_t)r * kBoxCells];
    int32_t sum = 0;
#pragma unroll
    for (int r = 0; r < kFoldReps; r++) {
      sum += v[r];
      if (v[r]) p[(size_t)r * kBoxCells] = 0;
    }
    const int dz = i % kBoxZ, t = i / kBoxZ;
    const int dy = t % kBoxXY, dx = t / kBoxXY;
    if (sum && dx < a.box_e[0] && dy < a.box_e[1] && dz < a.box_e[2]) {
      const int32_t sx = wrap_add(a.box_s[0] + dx, a.d.nx);
      const int32_t sy = wrap_add(a.box_s[1] + dy, a.d.ny);
      const int32_t sz = wrap_add(a.box_s[2] + dz, a.d.nz);
      const int32_t idx = col_base(a.d, sx, sy) + (sz << 4);
      atomicAdd(&a.passes[idx], sum);
      if (DISTINCT) {
        uint32_t* touch_p = a.touch + ((a.d.vs + 31) >> 5);
        const uint32_t bit = 1u << (idx & 31);
        const uint32_t old = atomicOr(&touch_p[(uint32_t)idx >> 5], bit);
        n_dpass = !(old & bit);
      }
    }
  }
  __shared__ int wsum[kBlock / 64];
  const int c = DISTINCT ? wave_sum(n_dpass) : 0;
  if (__lane_id() == 0) wsum[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long q = 0;
    for (int w = 0; w < kBlock / 64; w++) q += wsum[w];
    const size_t slot = (size_t)a.trace_blocks + by * kFoldCellBlocks + bx;
    unsigned long long* pt = a.part_trace + 4 * slot;
    pt[0] = 0;
    pt[1] = q;
    pt[2] = 0;
    pt[3] = 0;
  }
}

// Window scroll.  (One voxel per thread, three arrays and eight integer
// divisions for each, took 34 us for the slabs of a 1.2 m step on 1024 x 1024 x
// 96.)  The boxes' passes are zeroed in 16-byte words (four voxels of
// one brick row; words that reach past a box one voxel at a time); hits and
// lowest returns only where the columns' occupancy words have a voxel, then
// the words' bits.  The boxes of a column are combined by one thread, so that
// no two threads update one word.
__device__ __forceinline__ void clear_body(const ClearArgs& a, const int64_t first,
                                           const int64_t stride) {
  const Dims& d = a.d;
  if (a.nbox == 0) return;
  int k = 0;
  for (int64_t i = first; i < a.pre[a.nbox]; i += stride) {
    while (i >= a.pre[k + 1]) k++;
    const int32_t* b = a.box[k];
    // word (brick column bx, by, level z, brick row iy) of the box, in storage order
    const uint32_t nby = (uint32_t)((b[3] + 3) >> 2) - (uint32_t)(b[2] >> 2);
    const uint32_t nz = b[5] - b[4];
    const uint32_t w = (uint32_t)(i - a.pre[k]), t = w >> 2, u = t / nz;
    const int iy = w & 3, z = b[4] + (int)(t - u * nz);
    const int bx = (b[0] >> 2) + (int)(u / nby), by = (b[2] >> 2) + (int)(u % nby);
    const int sy = 4 * by + iy;
    if (sy < b[2] || sy >= b[3]) continue;
    int32_t* p = a.passes + col_base(d, 4 * bx, sy) + (z << 4);
    if (4 * bx >= b[0] && 4 * bx + 3 < b[1]) {
      *(int4*)p = make_int4(0, 0, 0, 0);
    } else {
#pragma unroll
      for (int ix = 0; ix < 4; ix++)
        if (4 * bx + ix >= b[0] && 4 * bx + ix < b[1]) p[ix] = 0;
    }
  }
  const auto clear_column = [&](int sx, int sy, unsigned long long k0, unsigned long long k1) {
    unsigned long long* o = a.occ + ((int64_t)sx * d.ny + sy) * d.W;
    const int32_t base = col_base(d, sx, sy);
    for (int h = 0; h < d.W; h++) {
      const unsigned long long keep = h ? k1 : k0, m = o[h];
      unsigned long long gone = m & ~keep;
      if (!gone) continue;
      o[h] = m & keep;
      while (gone) {
        const int32_t e = base + ((64 * h + __ffsll((long long)gone) - 1) << 4);
        gone &= gone - 1;
        a.hits[e] = 0;
        a.minqz[e] = INT32_MAX;
      }
    }
  };
  if (a.nslab < a.nbox) {  // some levels of every column go
    for (int64_t i = first; i < (int64_t)d.nx * d.ny; i += stride) {
      const int sx = (int)((uint32_t)i / (uint32_t)d.ny), sy = (int)((uint32_t)i % (uint32_t)d.ny);
      bool all = false;
      for (int j = 0; j < a.nslab; j++)
        all |= sx >= a.box[j][0] && sx < a.box[j][1] && sy >= a.box[j][2] && sy < a.box[j][3];
      clear_column(sx, sy, all ? 0ull : a.keep[0], all ? 0ull : a.keep[1]);
    }
  } else {
    // (a column of two slabs is emptied by both: the same stores)
    for (int j = 0; j < a.nslab; j++) {
      const uint32_t cy = a.box[j][3] - a.box[j][2];
      const int64_t cols = (int64_t)(a.box[j][1] - a.box[j][0]) * cy;
      for (int64_t i = first; i < cols; i += stride)
        clear_column(a.box[j][0] + (int)((uint32_t)i / cy), a.box[j][2] + (int)((uint32_t)i % cy),
                     0ull, 0ull);
    }
  }
}

}  // namespace
}  // namespace gvom
