// Host side of libgvom: the C ABI declared in include/gvom.h.  Validates
// arguments, owns the map state on the device, derives the host-side
// constants (sensor voxel, window origin, slabs to clear) and orders the
// kernel launches on the map's stream.  Nothing here waits on the device
// except where gvom.h says a call synchronises.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <stdio.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "gvom_internal.h"

using gvom::Dims;

#include "map_state.h"

namespace {

constexpr size_t kStatsBytes = (8 + gvom::kStripes) * 8;

int64_t n_vox(const map_t* m) { return (int64_t)m->p.nx * m->p.ny * m->p.nz; }
int64_t n_store(const map_t* m) { return m->d.vs; }
int64_t n_col(const map_t* m) { return (int64_t)m->p.nx * m->p.ny; }

int32_t pos_mod(int64_t a, int32_t n) {
  int64_t r = a % n;
  return (int32_t)(r < 0 ? r + n : r);
}

void set_ring(map_t* m) {
  m->d.ro[0] = pos_mod(m->origin[0], m->p.nx);
  m->d.ro[1] = pos_mod(m->origin[1], m->p.ny);
  m->d.ro[2] = pos_mod(m->origin[2], m->p.nz);
}

}  // namespace

namespace gvom {

namespace {
std::mutex g_mem_mu;
std::unordered_map<void*, size_t> g_mem_size;
int64_t g_mem_used = 0;
int64_t g_mem_cap = 0;  // 0: no cap
}  // namespace

hipError_t dev_alloc(void** p, size_t bytes) {
  *p = nullptr;
  std::lock_guard<std::mutex> lk(g_mem_mu);
  if (g_mem_cap > 0 && g_mem_used + (int64_t)bytes > g_mem_cap) return hipErrorOutOfMemory;
  const hipError_t e = hipMalloc(p, bytes);
  if (e != hipSuccess) {
    *p = nullptr;
    return e;
  }
  g_mem_size[*p] = bytes;
  g_mem_used += (int64_t)bytes;
  return hipSuccess;
}

hipError_t dev_free(void* p) {
  if (!p) return hipSuccess;
  {
    std::lock_guard<std::mutex> lk(g_mem_mu);
    auto it = g_mem_size.find(p);
    if (it != g_mem_size.end()) {
      g_mem_used -= (int64_t)it->second;
      g_mem_size.erase(it);
    }
  }
  return hipFree(p);
}

void set_origin(map_t* m, const int32_t o[3]) {
  for (int i = 0; i < 3; i++) m->origin[i] = o[i];
  set_ring(m);
}

void set_empty_origin(map_t* m, const int32_t o[3]) {
  if (m->empty) set_origin(m, o);
}

uint64_t capture_of(map_t* m) {
  if (!m->stream) return 0;  // the null stream is never captured
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  unsigned long long id = 0;
  if (hipStreamGetCaptureInfo(m->stream, &st, &id) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  if (st == hipStreamCaptureStatusNone) return 0;
  m->replays = true;
  return id;
}

uint64_t next_version() {
  static std::atomic<uint64_t> counter{0};
  return ++counter;
}

}  // namespace gvom

namespace {

int32_t dev_status(map_t* m, hipError_t e) {
  if (e != hipSuccess) {
    (void)hipGetLastError();
    m->sticky = MAP_E_DEVICE;
    return MAP_E_DEVICE;
  }
  return MAP_OK;
}

// Enqueues: every voxel empty, every occupancy word zero, whatever the memory
// holds.
hipError_t fill_all(map_t* m) {
  const int64_t V = n_store(m);
  hipError_t e = gvom::launch_fill_i32(m->hits, 0, V, m->stream);
  if (e == hipSuccess) e = gvom::launch_fill_i32(m->passes, 0, V, m->stream);
  if (e == hipSuccess) e = gvom::launch_fill_i32(m->minqz, INT32_MAX, V, m->stream);
  if (e == hipSuccess)
    e = gvom::launch_fill_i32((int32_t*)m->occ, 0, n_col(m) * m->d.W * 2, m->stream);
  return e;
}

// The same for a map whose occupancy words agree with its voxels (every map
// whose kernels all ran).
hipError_t clear_all(map_t* m) {
  return gvom::launch_thin(m->d, nullptr, m->hits, m->passes, m->minqz, m->occ, m->stream);
}

void initial_origin(map_t* m) {
  m->origin[0] = -m->p.nx / 2;
  m->origin[1] = -m->p.ny / 2;
  m->origin[2] = -m->p.sensor_z_voxel;
  set_ring(m);
}

// Moves the window to new origin `o` (whole voxels, Sec. III-A) and plans the
// clears of the storage slabs the new window takes over from the old one.
// Returns true when the whole window must be cleared.
bool move_window(map_t* m, const int32_t o[3], gvom::ClearArgs* plan) {
  const int32_t n[3] = {m->p.nx, m->p.ny, m->p.nz};
  int64_t delta[3];
  bool all = false;
  for (int a = 0; a < 3; a++) {
    delta[a] = (int64_t)o[a] - m->origin[a];
    if (delta[a] >= n[a] || -delta[a] >= n[a]) all = true;
  }
  plan->d = m->d;
  plan->hits = m->hits;
  plan->passes = m->passes;
  plan->minqz = m->minqz;
  plan->occ = m->occ;
  plan->nbox = 0;
  m->last_cleared = 0;
  if (delta[0] == 0 && delta[1] == 0 && delta[2] == 0) return false;
  for (int a = 0; a < 3; a++) m->origin[a] = o[a];
  set_ring(m);
  plan->d = m->d;
  plan->nslab = 0;
  plan->keep[0] = plan->keep[1] = ~0ull;
  plan->pre[0] = 0;
  // a box of storage range [s0, s1) along axis a (all of the other axes)
  const auto add_box = [&](int a, int32_t s0, int32_t s1) {
    int32_t* b = plan->box[plan->nbox];
    for (int k = 0; k < 3; k++) {
      b[2 * k] = k == a ? s0 : 0;
      b[2 * k + 1] = k == a ? s1 : n[k];
    }
    const int64_t words = (int64_t)(((b[1] + 3) >> 2) - (b[0] >> 2)) *
                          (((b[3] + 3) >> 2) - (b[2] >> 2)) * (b[5] - b[4]) * 4;
    plan->pre[plan->nbox + 1] = plan->pre[plan->nbox] + (int32_t)words;
    plan->nbox++;
    if (a < 2) plan->nslab++;
  };
  if (all) {
    m->last_cleared = n_vox(m);
    add_box(0, 0, n[0]);
    return true;
  }
  int64_t keep = 1;
  for (int a = 0; a < 3; a++) keep *= n[a] - (delta[a] < 0 ? -delta[a] : delta[a]);
  m->last_cleared = n_vox(m) - keep;
  for (int a = 0; a < 3; a++) {
    if (delta[a] == 0) continue;
    // storage range of the entering local range along axis a
    const int32_t s0 = delta[a] > 0 ? pos_mod((int64_t)n[a] - delta[a] + m->d.ro[a], n[a])
                                    : m->d.ro[a];
    const int32_t cnt = (int32_t)(delta[a] > 0 ? delta[a] : -delta[a]);
    // the range in one or, where it wraps, two pieces
    const int32_t s1 = s0 + cnt < n[a] ? s0 + cnt : n[a];
    add_box(a, s0, s1);
    if (s0 + cnt > n[a]) add_box(a, 0, s0 + cnt - n[a]);
    if (a == 2) {
      for (int j = 0; j < cnt; j++) {
        const int z = (s0 + j) % n[2];
        plan->keep[z >> 6] &= ~(1ull << (z & 63));
      }
    }
  }
  return false;
}

// Records the start event of a profiled phase (no-op when profiling is off).
int prof_begin(map_t* m, int phase) {
  if (!((m->prof_mask >> phase) & 1)) return -1;
  map_t::Mark k{phase, nullptr, nullptr};
  if (hipEventCreate(&k.a) != hipSuccess || hipEventCreate(&k.b) != hipSuccess) return -1;
  (void)hipEventRecord(k.a, m->stream);
  m->marks.push_back(k);
  return (int)m->marks.size() - 1;
}

void prof_end(map_t* m, int idx) {
  if (idx >= 0) (void)hipEventRecord(m->marks[idx].b, m->stream);
}

void prof_release(map_t* m) {
  for (auto& k : m->marks) {
    (void)hipEventDestroy(k.a);
    (void)hipEventDestroy(k.b);
  }
  m->marks.clear();
}

template <class T>
hipError_t dmalloc(T** p, size_t bytes) {
  return gvom::dev_alloc((void**)p, bytes < 16 ? 16 : bytes);
}

}  // namespace

extern "C" {

int32_t map_set_device_memory_limit(int64_t bytes) {
  if (bytes < 0) return MAP_E_INVALID;
  std::lock_guard<std::mutex> lk(gvom::g_mem_mu);
  gvom::g_mem_cap = bytes;
  return MAP_OK;
}

int64_t map_device_memory_in_use(void) {
  std::lock_guard<std::mutex> lk(gvom::g_mem_mu);
  return gvom::g_mem_used;
}

int32_t map_params_validate(const map_params_t* p, map_derived_t* out) {
  if (!p) return MAP_E_INVALID;
  if (p->nx < 2 || p->ny < 2 || p->nz < 1 || p->nx > 8192 || p->ny > 8192 || p->nz > 128)
    return MAP_E_INVALID;
  if ((p->nx & 1) || (p->ny & 1)) return MAP_E_INVALID;
  if ((int64_t)p->nx * p->ny * p->nz > 2147483647LL) return MAP_E_INVALID;
  if (!(p->res_m > 0.0f) || !isfinite(p->res_m)) return MAP_E_INVALID;
  if (p->sensor_z_voxel < 0 || p->sensor_z_voxel >= p->nz) return MAP_E_INVALID;
  if (!isfinite(p->obs_min_m) || !isfinite(p->obs_max_m) || p->obs_min_m < 0.0f ||
      p->obs_max_m < p->obs_min_m)
    return MAP_E_INVALID;
  if (p->dens_den <= 0 || p->dens_num < 0) return MAP_E_INVALID;
  if (p->fit_n < 3 || p->fit_n > 15 || !(p->fit_n & 1)) return MAP_E_INVALID;
  if (!isfinite(p->neg_thresh_m) || p->neg_thresh_m < 0.0f) return MAP_E_INVALID;
  if (!isfinite(p->neg_search_m) || p->neg_search_m < 0.0f) return MAP_E_INVALID;
  map_derived_t c;
  const double r = (double)p->res_m;
  c.inv_r = (float)(1.0 / r);
  const long lo = lround((double)p->obs_min_m / r);
  c.n_lo = (int32_t)(lo < 1 ? 1 : lo);
  c.n_hi = (int32_t)lround((double)p->obs_max_m / r);
  c.tau_neg_q = (int64_t)floor((double)p->neg_thresh_m / r * 65536.0);
  c.search_d = (int32_t)lround((double)p->neg_search_m / r);
  c.half_fit = (p->fit_n - 1) / 2;
  if (c.n_hi < c.n_lo) return MAP_E_INVALID;
  if (c.search_d < 1 || c.search_d > 64) return MAP_E_INVALID;
  if (out) *out = c;
  return MAP_OK;
}

int32_t map_create(const map_params_t* p, void* stream, map_t** out) {
  if (!out) return MAP_E_INVALID;
  *out = nullptr;
  map_derived_t c;
  int32_t s = map_params_validate(p, &c);
  if (s) return s;
  map_t* m = new (std::nothrow) map_t();
  if (!m) return MAP_E_OOM;
  m->p = *p;
  m->c = c;
  m->stream = (hipStream_t)stream;
  if (hipGetDevice(&m->device) != hipSuccess ||
      hipDeviceGetAttribute(&m->n_cu, hipDeviceAttributeMultiprocessorCount, m->device) !=
          hipSuccess) {
    delete m;
    return MAP_E_DEVICE;
  }
  m->seg_len = 8;
  m->trace_wpc = 28;
  m->surf_tile = 32;
  m->seg_auto = m->tile_auto = true;
  // traversal blocks (at most 32 waves per CU) + the sensor-box fold blocks
  m->part_trace_cap = (int64_t)m->n_cu * 32 / 4 + gvom::box_fold_blocks() + 1;
  m->d.nx = p->nx;
  m->d.ny = p->ny;
  m->d.nz = p->nz;
  m->d.W = (p->nz + 63) / 64;
  m->d.nby = (p->ny + 3) / 4;
  m->d.vs = (int64_t)((p->nx + 3) / 4) * m->d.nby * p->nz * 16;
  if (m->d.vs > 2147483647LL) {  // the 4-aligned storage must stay int32-indexable
    delete m;
    return MAP_E_INVALID;
  }
  const int64_t V = n_store(m), C = n_col(m);
  const int64_t nb = (C + 63) / 64;
  hipError_t e = dmalloc(&m->hits, V * 4);
  if (e == hipSuccess) e = dmalloc(&m->passes, V * 4);
  if (e == hipSuccess) e = dmalloc(&m->minqz, V * 4);
  if (e == hipSuccess) e = dmalloc(&m->occ, C * m->d.W * 8);
  if (e == hipSuccess) e = dmalloc(&m->hq, C * 4);
  if (e == hipSuccess) e = dmalloc(&m->defbits, nb * 8);
  if (e == hipSuccess) e = dmalloc(&m->group_cnt, nb * 4);
  if (e == hipSuccess) e = dmalloc(&m->colpre, C * 4);
  if (e == hipSuccess) e = dmalloc(&m->super_sum, (nb + 63) / 64 * 4);
  if (e == hipSuccess) e = dmalloc(&m->stats, kStatsBytes);
  if (e == hipSuccess) e = dmalloc(&m->imported, 4);
  if (e == hipSuccess) e = dmalloc(&m->nocc, 8);
  if (e == hipSuccess) e = hipHostMalloc((void**)&m->host, 8, 0);
  if (e == hipSuccess) e = dmalloc(&m->part_trace, m->part_trace_cap * 32);
  if (e == hipSuccess) e = dmalloc(&m->box_rep, (int64_t)gvom::kBoxReps * gvom::kBoxCells * 4);
  if (e == hipSuccess)
    e = hipMemsetAsync(m->box_rep, 0, (size_t)gvom::kBoxReps * gvom::kBoxCells * 4, m->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    map_destroy(m);
    return MAP_E_OOM;
  }
  initial_origin(m);
  e = fill_all(m);
  m->empty = true;
  m->version = gvom::next_version();
  if (e == hipSuccess) e = hipMemsetAsync(m->stats, 0, kStatsBytes, m->stream);
  if (e == hipSuccess) e = hipMemsetAsync(m->imported, 0, 4, m->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    map_destroy(m);
    return MAP_E_DEVICE;
  }
  *out = m;
  return MAP_OK;
}

int32_t map_destroy(map_t* m) {
  if (!m) return MAP_OK;
  (void)hipStreamSynchronize(m->stream);
  prof_release(m);
  (void)gvom::dev_free(m->hits);
  (void)gvom::dev_free(m->passes);
  (void)gvom::dev_free(m->minqz);
  (void)gvom::dev_free(m->occ);
  (void)gvom::dev_free(m->hq);
  (void)gvom::dev_free(m->defbits);
  (void)gvom::dev_free(m->group_cnt);
  (void)gvom::dev_free(m->colpre);
  (void)gvom::dev_free(m->super_sum);
  (void)gvom::dev_free(m->stats);
  (void)gvom::dev_free(m->imported);
  (void)gvom::dev_free(m->nocc);
  (void)hipHostFree(m->host);
  (void)gvom::dev_free(m->touch);
  (void)gvom::dev_free(m->rays);
  (void)gvom::dev_free(m->witems);
  (void)gvom::dev_free(m->part_rays);
  (void)gvom::dev_free(m->part_trace);
  (void)gvom::dev_free(m->box_rep);
  delete m;
  return MAP_OK;
}

int32_t map_reset(map_t* m) {
  if (!m) return MAP_E_INVALID;
  // after an error the kernels that keep voxels and occupancy words in step
  // may not have run
  const bool intact = hipStreamSynchronize(m->stream) == hipSuccess && m->sticky == MAP_OK;
  (void)hipGetLastError();
  m->sticky = MAP_OK;
  initial_origin(m);
  m->ranked = false;
  m->version = gvom::next_version();
  m->last_points = 0;
  m->last_cleared = 0;
  m->last_distinct = false;
  m->last_ray_blocks = 0;
  m->last_trace_blocks = 0;
  hipError_t e = intact ? clear_all(m) : fill_all(m);
  m->empty = true;
  const bool told = m->wild || !intact;  // the import's word may not be zero
  m->wild = false;
  if (e == hipSuccess) e = hipMemsetAsync(m->stats, 0, kStatsBytes, m->stream);
  if (e == hipSuccess && told) e = hipMemsetAsync(m->imported, 0, 4, m->stream);
  // an insert that failed between the traversal and the fold leaves counts
  if (e == hipSuccess)
    e = hipMemsetAsync(m->box_rep, 0, (size_t)gvom::kBoxReps * gvom::kBoxCells * 4, m->stream);
  return dev_status(m, e);
}

}  // extern "C"

namespace {

// Checks an insert request without changing anything; derives the sensor Q.
int32_t check_insert(const map_t* m, const float* xyz_dev, int64_t n, const float* pose,
                     uint32_t flags, int32_t S[3]) {
  if (!m || !pose || n < 0 || n > 2147483647LL || (n > 0 && !xyz_dev)) return MAP_E_INVALID;
  if (flags & 0x0000FFFCu) return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  for (int i = 0; i < 12; i++)
    if (!isfinite(pose[i])) return MAP_E_POSE;
  for (int i = 0; i < 3; i++) {
    const float u = pose[4 * i + 3] * m->c.inv_r;
    if (!(fabsf(u) < 32768.0f)) return MAP_E_RANGE;
    S[i] = (int32_t)floorf(u * 65536.0f);
  }
  if (!(flags & MAP_RECENTER)) {
    const int32_t n3[3] = {m->p.nx, m->p.ny, m->p.nz};
    for (int a = 0; a < 3; a++) {
      const int64_t l = (int64_t)(S[a] >> 16) - m->origin[a];
      if (l < 0 || l >= n3[a]) return MAP_E_SENSOR_OUTSIDE;
    }
  }
  return MAP_OK;
}

// Grows a device buffer (synchronising first); false on allocation failure.
// A regrow at least doubles the capacity (exactly `need` if that fails), so
// scans of growing size reallocate O(log) times: a free synchronises the
// device and would otherwise stall every step that sees a new largest scan.
template <class T>
bool grow(map_t* m, T** p, int64_t* cap, int64_t need, size_t elem) {
  if (need <= *cap) return true;
  if (hipStreamSynchronize(m->stream) != hipSuccess) return false;
  const int64_t want = *cap > 0 && need < 2 * *cap ? 2 * *cap : need;
  (void)gvom::dev_free(*p);
  *p = nullptr;
  *cap = 0;
  if (dmalloc(p, (size_t)want * elem) == hipSuccess) {
    *cap = want;
    return true;
  }
  (void)hipGetLastError();
  *p = nullptr;
  if (want > need && dmalloc(p, (size_t)need * elem) == hipSuccess) {
    *cap = need;
    return true;
  }
  (void)hipGetLastError();
  *p = nullptr;
  return false;
}

// The wave-item regions of the ray pass: ray block b reserves its waves'
// items in the region of stripe b mod kStripes, sized for the most items
// that stripe's waves can reserve (each wave at most one item per segment
// its longest ray can have).  *need = wave items in all.
void insert_layout(const map_t* m, int64_t ray_blocks, int32_t seg_len, gvom::InsertArgs* a,
                   int64_t* need) {
  a->seg_len = seg_len;
  a->block_items = (gvom::kRayBlock / 64) * gvom::max_segments(m->d, seg_len);
  *need = ray_blocks * a->block_items;
}

// Segment length of a lone insert of n points, where none was set.  An item's steps are
// one chain of LDS round trips, so a scan with fewer items than the device has waves
// ends sooner when its rays are cut shorter; with more items their set-up and the flush
// of their lines cost more than the chains.  The items grow with the points and with the
// voxels a ray can cross (n x the window's longer side); on windows beyond 512 a far
// segment has most lines to itself, so cutting it again adds flushes.  Whole insert with
// 4 / 5 / 8 voxels (events included), 64-beam scans and every k-th point of them:
//   256 x 256 x 48: 65,536 points 34.4 / 35.2 / 37.3 us, 131,072 50.6 / 48.7 / 51.2,
//     196,608 66.9 / 62.5 / 63.0, 262,144 81.8 / 77.8 / 76.6
//   512 x 512 x 64: 32,768 31.5 / 31.5 / 34.4, 65,536 46.7 / 43.4 / 44.5, 131,072 75.1 /
//     74.8 / 77.1, 196,608 95.8 / 94.4 / 97.5, 262,144 125.3 / 123.4 / 123.9
//   1024 x 1024 x 96: 16,384 32.6 / 32.7 / 36.8, 32,768 44.6 / 40.9 / 39.6, 49,152 60.2 /
//     55.9 / 54.3, 131,072 132 / 133 / 134, 196,608 175 / 166 / 159
//   4096 x 4096 x 4, short rays: 5,000 30.7 / - / 36.9 (beyond 1024 a window is longer
//     than most rays, so it counts as 1024)
// (The shorter segments cost traffic: at 131,072 points on 512 x 512 x 64 the traversal
// makes 0.311 M line requests and moves 26.4 MB with 5, 0.265 M and 23.8 MB with 8.)  In a
// batch the maps fill the device together: 8.
int32_t lone_seg_len(const map_t* m, int64_t n) {
  const int64_t side = std::max(m->p.nx, m->p.ny);
  if (!m->seg_auto) return m->seg_len;
  if (n * std::min<int64_t>(side, 1024) <= (int64_t)1 << 24) return 4;
  return side <= 512 && n <= 196608 ? 5 : m->seg_len;
}

// Everything of an insert but the per-scan buffers (a->rays, a->witems,
// a->part_rays, set by the caller).
int32_t fill_insert(map_t* m, const float* xyz_dev, int64_t n, const float* pose,
                    uint32_t flags, const int32_t S[3], gvom::InsertArgs* a,
                    gvom::ClearArgs* plan, bool* full, int64_t need) {
  const int64_t ray_blocks = (n + gvom::kRayBlock - 1) / gvom::kRayBlock;
  *full = false;
  plan->nbox = 0;
  if (flags & MAP_RECENTER) {
    const int32_t o[3] = {(S[0] >> 16) - m->p.nx / 2, (S[1] >> 16) - m->p.ny / 2,
                          (S[2] >> 16) - m->p.sensor_z_voxel};
    *full = move_window(m, o, plan);
  } else {
    m->last_cleared = 0;
  }
  m->last_points = n;
  m->last_distinct = false;
  m->last_static = false;
  m->last_ray_blocks = n > 0 ? ray_blocks : 0;
  a->xyz = xyz_dev;
  a->n = (int32_t)n;
  uint32_t fw = flags >> 16;
  if (fw < 1 || (n > 0 && n % fw != 0)) fw = 1;
  a->fw = (int32_t)fw;
  a->azimuths = (int32_t)(n / fw);
  for (int i = 0; i < 3; i++) {
    for (int j = 0; j < 3; j++) a->R[3 * i + j] = pose[4 * i + j];
    a->t[i] = pose[4 * i + 3];
    a->S[i] = S[i];
    a->O[i] = m->origin[i];
  }
  a->inv_r = m->c.inv_r;
  a->d = m->d;
  a->hits = m->hits;
  a->passes = m->passes;
  a->minqz = m->minqz;
  a->occ = m->occ;
  a->stats = m->stats;
  a->touch = m->touch;
  a->part_trace = m->part_trace;
  const int64_t tpb = gvom::kTraceBlock;  // threads per traversal block
  const int64_t want = (need + tpb / 64 - 1) / (tpb / 64);  // one wave per item
  int64_t lim = (int64_t)m->n_cu * m->trace_wpc / (tpb / 64);
  if (lim < 1) lim = 1;
  a->trace_blocks = n > 0 ? (int32_t)(want < lim ? want : lim) : 0;
  // sensor box of the segmented traversal: the box of kBoxXY x kBoxXY x kBoxZ
  // window cells centred on the sensor's voxel, moved inside the window
  const int32_t ext[3] = {gvom::kBoxXY, gvom::kBoxXY, gvom::kBoxZ};
  const int32_t dims[3] = {m->d.nx, m->d.ny, m->d.nz};
  a->box_far = 0;
  for (int k = 0; k < 3; k++) {
    const int32_t e = ext[k] < dims[k] ? ext[k] : dims[k];
    int64_t lo = (int64_t)(S[k] >> 16) - m->origin[k] - ext[k] / 2;
    if (lo > dims[k] - e) lo = dims[k] - e;
    if (lo < 0) lo = 0;
    a->box_e[k] = e;
    const int64_t l = (int64_t)(S[k] >> 16) - m->origin[k];
    const int64_t far = l - lo > lo + e - 1 - l ? l - lo : lo + e - 1 - l;
    if (far > a->box_far) a->box_far = (int32_t)far;
    a->box_s[k] = (int32_t)((lo + m->d.ro[k]) % dims[k]);
  }
  a->box_rep = m->box_rep;
  m->last_trace_blocks = a->trace_blocks + gvom::box_fold_blocks();
  if (n <= 0) m->last_trace_blocks = 0;
  return MAP_OK;
}

// Second half of an insert (after check_insert): grows the per-scan buffers,
// moves the window (the slab clears go to `plan`; *full = whole window), and
// fills the kernel arguments.  Updates the host-side map state.
int32_t prepare_insert(map_t* m, const float* xyz_dev, int64_t n, const float* pose,
                       uint32_t flags, const int32_t S[3], gvom::InsertArgs* a,
                       gvom::ClearArgs* plan, bool* full, int32_t seg_len) {
  const int64_t ray_blocks = (n + gvom::kRayBlock - 1) / gvom::kRayBlock;
  int64_t need = 0;
  if (!grow(m, &m->rays, &m->rays_cap, ray_blocks * gvom::kRayBlock, sizeof(int4)))
    return MAP_E_OOM;
  // Where the items of shorter segments find no room, the setting's length; and as
  // long as the buffer holds that one's items, no growing is tried again (each try
  // waits for the stream, frees the buffer and allocates).
  const auto fits = [&](int32_t len) {
    insert_layout(m, ray_blocks, len, a, &need);
    return need <= m->witem_cap;
  };
  if (seg_len != m->seg_len && !fits(seg_len) && m->short_oom && need >= m->short_oom &&
      fits(m->seg_len))
    seg_len = m->seg_len;
  if (!fits(seg_len) && !grow(m, &m->witems, &m->witem_cap, need, sizeof(int2))) {
    if (seg_len == m->seg_len) return MAP_E_OOM;
    m->short_oom = need;
    if (!fits(m->seg_len) && !grow(m, &m->witems, &m->witem_cap, need, sizeof(int2)))
      return MAP_E_OOM;
  }
  if (!grow(m, &m->part_rays, &m->part_rays_cap, ray_blocks, 32)) return MAP_E_OOM;
  a->rays = m->rays;
  a->witems = m->witems;
  a->part_rays = m->part_rays;
  return fill_insert(m, xyz_dev, n, pose, flags, S, a, plan, full, need);
}

// ranks: also write the table export's per-column ranks (in a batch where it exports
// the map's table)
void column_args(const map_t* m, const map_2d_t* out, bool ranks, gvom::ColumnArgs* ca) {
  ca->d = m->d;
  ca->hits = m->hits;
  ca->passes = m->passes;
  ca->minqz = m->minqz;
  ca->occ = m->occ;
  ca->res = (double)m->p.res_m;
  ca->n_lo = m->c.n_lo;
  ca->n_hi = m->c.n_hi;
  ca->dens_num = m->p.dens_num;
  ca->dens_den = m->p.dens_den;
  ca->height = out->height;
  ca->density = out->density;
  ca->flags = out->flags;
  ca->hq = m->hq;
  ca->defbits = m->defbits;
  ca->colpre = ranks ? m->colpre : nullptr;
  ca->group_cnt = ranks ? m->group_cnt : nullptr;
}

int64_t tiles64(const map_t* m) {
  return (int64_t)((m->p.nx + 63) / 64) * ((m->p.ny + 63) / 64);
}

int32_t surf_halo(const map_t* m) {
  return m->c.search_d > m->c.half_fit ? m->c.search_d : m->c.half_fit;
}

// Tile edge of the surface pass in a launch of t64 64-pixel tiles.
int32_t surf_tile(const map_t* m, int64_t t64) {
  return m->tile_auto ? gvom::surface_tile_for(surf_halo(m), t64, m->n_cu) : m->surf_tile;
}

// ranks: the launch also sums the group counts of the column pass
void surface_args(const map_t* m, const map_2d_t* out, bool ranks, gvom::SurfaceArgs* sa) {
  sa->rank_cnt = m->group_cnt;
  sa->rank_n = ranks ? (int32_t)((n_col(m) + 63) / 64) : 0;
  sa->rank_sum = m->super_sum;
  sa->nx = m->p.nx;
  sa->ny = m->p.ny;
  sa->hq = m->hq;
  sa->defbits = (const uint32_t*)m->defbits;
  sa->imported = m->imported;
  sa->half_fit = m->c.half_fit;
  sa->search_d = m->c.search_d;
  sa->tau_q = m->c.tau_neg_q;
  sa->q2m = (double)m->p.res_m / 65536.0;
  sa->slope = out->slope;
  sa->rough = out->rough;
  sa->flags = out->flags;
}

void lut_args(const map_t* m, int32_t* lut_dev, map_voxel_t* data_dev, int64_t cap,
              int64_t* n_occupied_dev, gvom::LutArgs* a) {
  a->d = m->d;
  a->hits = m->hits;
  a->passes = m->passes;
  a->minqz = m->minqz;
  a->occ = m->occ;
  a->lut = lut_dev;
  a->data = data_dev;
  a->cap = cap;
  a->group_cnt = m->group_cnt;
  a->colpre = m->colpre;
  a->super_sum = m->super_sum;
  a->nsuper = (int32_t)((n_col(m) + 4095) / 4096);
  a->scanned = 0;
  a->n_occupied = n_occupied_dev;
}

bool valid_2d(const map_2d_t* out) {
  return out && out->height && out->slope && out->rough && out->density && out->flags;
}

}  // namespace

// ---- the insert without allocation (map_insert_scan_static) ----------------
// Its per-scan work buffers (ray records, wave items, per-block ray counters)
// live in this file-scope device array instead of buffers the map grows: one
// copy per device, held until the process ends, shared by every such call on
// that device.
constexpr size_t kScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxDevices];  // device address of `scratch`, per device

// Device address of the scratch array on device `dev`, looked up once per
// device with that device current (the array's host-side name is not a
// device address); null on failure.
unsigned char* device_scratch(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess) return nullptr;
    if (cur != dev && hipSetDevice(dev) != hipSuccess) return nullptr;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = (unsigned char*)p;
  }
  return g_scratch_ptr[dev];
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Bytes of the scratch an insert of n points needs (ray records, wave items,
// per-block counters), each region 256-byte aligned.
size_t static_insert_bytes(const map_t* m, int64_t n, int32_t seg_len, int64_t* need) {
  const int64_t ray_blocks = (n + gvom::kRayBlock - 1) / gvom::kRayBlock;
  gvom::InsertArgs tmp;
  insert_layout(m, ray_blocks, seg_len, &tmp, need);
  return align256((size_t)ray_blocks * gvom::kRayBlock * sizeof(int4)) +
         align256((size_t)*need * sizeof(int2)) + align256((size_t)ray_blocks * 32);
}

}  // namespace

extern "C" {

int32_t map_insert_scan(map_t* m, const float* xyz_dev, int64_t n, const float pose[12],
                        uint32_t flags) {
  int32_t S[3];
  int32_t st = check_insert(m, xyz_dev, n, pose, flags, S);
  if (st) return st;
  gvom::InsertArgs a;
  gvom::ClearArgs plan;
  bool full = false;
  (void)gvom::capture_of(m);
  m->ranked = false;
  m->version = gvom::next_version();
  const int pm0 = prof_begin(m, MAP_PROF_SCROLL);
  st = prepare_insert(m, xyz_dev, n, pose, flags, S, &a, &plan, &full, lone_seg_len(m, n));
  if (st) return st;
  // an empty map moves its window without clearing anything; the slabs of a
  // moved one are cleared beside the ray pass
  hipError_t e = hipSuccess;
  if (m->empty || full) plan.nbox = 0;
  if (full && !m->empty) e = clear_all(m);
  if (n > 0) m->empty = false;
  prof_end(m, pm0);
  const bool distinct = (flags & MAP_STATS_DISTINCT) != 0;
  m->last_distinct = distinct;
  // the segment counters of stats start at zero: zeroed at creation and by
  // the sensor-box fold that ends every insert with points
  if (distinct && e == hipSuccess) {
    const int64_t words = (n_store(m) + 31) / 32;
    if (!m->touch) e = dmalloc(&m->touch, words * 2 * 4);
    if (e == hipSuccess) e = hipMemsetAsync(m->touch, 0, words * 2 * 4, m->stream);
    a.touch = m->touch;
  }
  if (e == hipSuccess && n == 0) e = gvom::launch_clear(plan, m->stream);
  if (e == hipSuccess && n > 0) {
    int pm = prof_begin(m, MAP_PROF_RAYS);
    e = gvom::launch_rays(a, plan, m->stream);
    prof_end(m, pm);
    if (e == hipSuccess) {
      pm = prof_begin(m, MAP_PROF_TRACE);
      e = gvom::launch_trace(a, distinct, m->stream);
      prof_end(m, pm);
    }
  }
  return dev_status(m, e);
}

int32_t map_insert_scan_static(map_t* m, const float* xyz_dev, int64_t n, const float pose[12],
                               uint32_t flags) {
  int32_t S[3];
  if (m && (flags & MAP_STATS_DISTINCT)) return MAP_E_INVALID;
  int32_t st = check_insert(m, xyz_dev, n, pose, flags, S);
  if (st) return st;
  int64_t need = 0;
  // (shorter segments of the library's choice always fit: 6 MB at most)
  const int32_t seg_len = lone_seg_len(m, n);
  if (static_insert_bytes(m, n, seg_len, &need) > kScratchBytes) return MAP_E_CAPACITY;
  unsigned char* base = device_scratch(m->device);
  if (!base) return MAP_E_DEVICE;  // nothing enqueued, the map is unchanged
  gvom::InsertArgs a;
  gvom::ClearArgs plan;
  bool full = false;
  const int64_t ray_blocks = (n + gvom::kRayBlock - 1) / gvom::kRayBlock;
  insert_layout(m, ray_blocks, seg_len, &a, &need);
  a.rays = (int4*)base;
  base += align256((size_t)ray_blocks * gvom::kRayBlock * sizeof(int4));
  a.witems = (int2*)base;
  base += align256((size_t)need * sizeof(int2));
  a.part_rays = (unsigned long long*)base;
  (void)gvom::capture_of(m);
  m->ranked = false;
  m->version = gvom::next_version();
  st = fill_insert(m, xyz_dev, n, pose, flags, S, &a, &plan, &full, need);
  if (st) return st;
  m->last_static = true;
  // kernels only (no memset, no allocation): callers may capture this call
  hipError_t e = hipSuccess;
  if (m->empty || full) plan.nbox = 0;
  if (full && !m->empty) e = clear_all(m);
  if (n > 0) m->empty = false;
  if (e == hipSuccess && n == 0) e = gvom::launch_clear(plan, m->stream);
  if (e == hipSuccess)
    e = gvom::launch_fill_i32((int32_t*)m->stats, 0, (int64_t)(kStatsBytes / 4), m->stream);
  if (e == hipSuccess && n > 0) {
    e = gvom::launch_rays(a, plan, m->stream);
    if (e == hipSuccess) e = gvom::launch_trace(a, false, m->stream);
    if (e == hipSuccess) e = gvom::launch_sum_ray_parts(a.part_rays, ray_blocks, m->stats, m->stream);
  }
  return dev_status(m, e);
}

int32_t map_export_2d(map_t* m, const map_2d_t* out) {
  if (!m || !valid_2d(out)) return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  m->rank_capture = gvom::capture_of(m);
  gvom::ColumnArgs ca;
  column_args(m, out, true, &ca);
  int pm = prof_begin(m, MAP_PROF_COLUMN);
  hipError_t e = gvom::launch_column(ca, m->stream);
  prof_end(m, pm);
  if (e == hipSuccess) {
    gvom::SurfaceArgs sa;
    surface_args(m, out, true, &sa);
    pm = prof_begin(m, MAP_PROF_SURFACE);
    e = gvom::launch_surface(sa, surf_tile(m, tiles64(m)), m->stream);
    prof_end(m, pm);
    m->ranked = e == hipSuccess;
  }
  return dev_status(m, e);
}

int32_t map_export_voxels_async(map_t* m, int32_t* lut_dev, map_voxel_t* data_dev, int64_t cap,
                                int64_t* n_occupied_dev, int32_t origin_vox[3]) {
  if (!m || !lut_dev || !n_occupied_dev || !origin_vox || cap < 0 || (cap > 0 && !data_dev))
    return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  gvom::LutArgs a;
  lut_args(m, lut_dev, data_dev, cap, n_occupied_dev, &a);
  const int pm = prof_begin(m, MAP_PROF_LUT);
  // The ranks of a 2D export since the last change of the map are used once, and only
  // where both exports run together: both captured into one graph, or neither in any
  // and no call on the map ever captured (a replay between them, which the host does
  // not see, may change the map or the ranks).  Any other export makes its own.
  const uint64_t capture = gvom::capture_of(m);
  const bool ranked = m->ranked && capture == m->rank_capture && (capture || !m->replays);
  hipError_t e = gvom::launch_lut(a, ranked, m->stream);
  m->ranked = false;
  prof_end(m, pm);
  for (int i = 0; i < 3; i++) origin_vox[i] = m->origin[i];
  return dev_status(m, e);
}

int32_t map_export_voxels(map_t* m, int32_t* lut_dev, map_voxel_t* data_dev, int64_t cap,
                          int64_t* n_occupied, int32_t origin_vox[3]) {
  if (!m || !n_occupied) return MAP_E_INVALID;
  int32_t s = map_export_voxels_async(m, lut_dev, data_dev, cap, m->nocc, origin_vox);
  if (s) return s;
  hipError_t e = hipMemcpyAsync(m->host, m->nocc, 8, hipMemcpyDeviceToHost, m->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  s = dev_status(m, e);
  if (s) return s;
  const int64_t count = *m->host;
  *n_occupied = count;
  return count > cap ? MAP_E_CAPACITY : MAP_OK;
}

int32_t map_export_density(map_t* m, float* density_dev) {
  if (!m || !density_dev) return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  gvom::DensityArgs a;
  a.d = m->d;
  a.hits = m->hits;
  a.passes = m->passes;
  a.occ = m->occ;
  a.out = density_dev;
  return dev_status(m, gvom::launch_density(a, m->stream));
}

int32_t map_costmap(map_t* m, const map_2d_t* in_dev, const map_cost_weights_t* w,
                    float* cost_dev) {
  if (!m || !valid_2d(in_dev) || !w || !cost_dev) return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  const float wv[8] = {w->slope, w->rough, w->density, w->positive,
                       w->hard, w->soft, w->negative, w->unknown};
  gvom::CostArgs a;
  for (int i = 0; i < 8; i++) {
    if (!isfinite(wv[i])) return MAP_E_INVALID;
    a.w[i] = wv[i];
  }
  a.n = n_col(m);
  a.slope = in_dev->slope;
  a.rough = in_dev->rough;
  a.density = in_dev->density;
  a.flags = in_dev->flags;
  a.cost = cost_dev;
  return dev_status(m, gvom::launch_costmap(a, m->stream));
}

int32_t map_import_voxels(map_t* m, const int32_t* lut_dev, const map_voxel_t* data_dev,
                          int64_t n_data, const int32_t origin_vox[3]) {
  if (!m || !lut_dev || !origin_vox || n_data < 0 || (n_data > 0 && !data_dev))
    return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  for (int i = 0; i < 3; i++) m->origin[i] = origin_vox[i];
  set_ring(m);
  m->ranked = false;
  m->empty = false;
  m->version = gvom::next_version();
  hipError_t e = hipMemsetAsync(m->imported, 0, 4, m->stream);
  if (e == hipSuccess)
    e = gvom::launch_import(m->d, lut_dev, data_dev, n_data, m->hits, m->passes, m->minqz,
                            m->occ, m->origin[2], m->imported, m->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(m->host, m->imported, 4, hipMemcpyDeviceToHost, m->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess) return dev_status(m, e);
  const int32_t err = *(const int32_t*)m->host;
  m->wild = (err & gvom::kWild) != 0;
  if (err & gvom::kBadContent) {
    m->wild = false;
    initial_origin(m);
    e = clear_all(m);
    if (e == hipSuccess) e = hipMemsetAsync(m->imported, 0, 4, m->stream);
    m->empty = true;
    if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
    if (e != hipSuccess) return dev_status(m, e);
    return MAP_E_INVALID;
  }
  return MAP_OK;
}

int32_t map_get_stats(map_t* m, map_stats_t* out) {
  if (!m || !out) return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  // a static insert left its ray-pass sums in stats[0..3] (one "block")
  const int64_t nrb = m->last_static ? (m->last_ray_blocks ? 1 : 0) : m->last_ray_blocks;
  std::vector<unsigned long long> pr((size_t)nrb * 4 + 1),
      pt((size_t)m->last_trace_blocks * 4 + 1);
  hipError_t e = hipSuccess;
  if (nrb)
    e = hipMemcpyAsync(pr.data(), m->last_static ? m->stats : m->part_rays, nrb * 32,
                       hipMemcpyDeviceToHost, m->stream);
  if (e == hipSuccess && m->last_trace_blocks)
    e = hipMemcpyAsync(pt.data(), m->part_trace, m->last_trace_blocks * 32,
                       hipMemcpyDeviceToHost, m->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess) return dev_status(m, e);
  int64_t c[7] = {0, 0, 0, 0, 0, 0, 0};
  for (int64_t b = 0; b < nrb; b++) {
    c[0] += (int64_t)pr[4 * b + 0];
    c[1] += (int64_t)pr[4 * b + 1];
    c[2] += (int64_t)pr[4 * b + 2];
  }
  for (int64_t b = 0; b < m->last_trace_blocks; b++) {
    c[3] += (int64_t)pt[4 * b + 0];
    c[4] += (int64_t)pt[4 * b + 1];
    c[6] += (int64_t)pt[4 * b + 2];
    c[5] += (int64_t)pt[4 * b + 3];
  }
  out->n_points = m->last_points;
  out->n_nonfinite = c[0];
  out->n_range = c[1];
  out->n_hits = c[2];
  out->n_pass = c[3];
  out->n_distinct_pass = m->last_distinct ? c[4] : -1;
  out->n_distinct_hit = m->last_distinct ? c[5] : -1;
  out->n_cleared = m->last_cleared;
  out->n_pass_updates = c[6];
  return MAP_OK;
}

int32_t map_get_origin(const map_t* m, int32_t origin_vox[3]) {
  if (!m || !origin_vox) return MAP_E_INVALID;
  for (int i = 0; i < 3; i++) origin_vox[i] = m->origin[i];
  return MAP_OK;
}

int32_t map_sync(map_t* m) {
  if (!m) return MAP_E_INVALID;
  if (m->sticky) return m->sticky;
  return dev_status(m, hipStreamSynchronize(m->stream));
}

int32_t map_set_tuning(map_t* m, const map_tuning_t* t) {
  if (!m || !t) return MAP_E_INVALID;
  if (t->seg_len > 1024 || t->trace_waves_per_cu > 32) return MAP_E_INVALID;
  if (!(t->surface_tile <= 0 || t->surface_tile == 16 || t->surface_tile == 32))
    return MAP_E_INVALID;
  // the wave-item buffer is sized for the segment length at the next insert
  if (t->seg_len > 0) {
    m->seg_len = t->seg_len;
    m->seg_auto = false;
  }
  if (t->trace_waves_per_cu > 0) m->trace_wpc = t->trace_waves_per_cu;
  if (t->surface_tile > 0) {
    m->surf_tile = t->surface_tile;
    m->tile_auto = false;
  }
  return MAP_OK;
}

int32_t map_get_tuning(const map_t* m, map_tuning_t* out) {
  if (!m || !out) return MAP_E_INVALID;
  out->seg_len = m->seg_len;
  out->trace_waves_per_cu = m->trace_wpc;
  out->surface_tile = m->surf_tile;
  return MAP_OK;
}

int32_t map_profile_enable(map_t* m, int32_t phase_mask) {
  if (!m || phase_mask < 0 || phase_mask > MAP_PROF_ALL) return MAP_E_INVALID;
  m->prof_mask = phase_mask;
  return MAP_OK;
}

int32_t map_profile_read(map_t* m, double ms[MAP_PROF_N], int64_t count[MAP_PROF_N]) {
  if (!m || !ms || !count) return MAP_E_INVALID;
  hipError_t e = hipStreamSynchronize(m->stream);
  if (e != hipSuccess) return dev_status(m, e);
  for (auto& k : m->marks) {
    float t = 0.0f;
    if (hipEventElapsedTime(&t, k.a, k.b) == hipSuccess) {
      ms[k.phase] += t;
      count[k.phase] += 1;
    }
  }
  prof_release(m);
  return MAP_OK;
}

// ---- batches ---------------------------------------------------------------

}  // extern "C"

struct map_batch_t {
  int k;
  map_t* maps[gvom::kMaxBatch];
  hipStream_t stream;
  int device, n_cu;
  gvom::BatchTables* dtab;
  gvom::BatchTables* htab;  // pinned
  unsigned long long* dstamps;
  unsigned long long* hstamps;  // pinned
  gvom::BatchGrid grid;
  bool use_graph, captured;
  hipGraph_t graph;
  hipGraphExec_t exec;
  bool own_stream;
  double clock_khz;
  double last_ms[gvom::kMaxBatch];
};

namespace {

hipError_t enqueue_batch(map_batch_t* b) {
  hipError_t e = hipMemcpyAsync(b->dtab, b->htab, sizeof(gvom::BatchTables),
                                hipMemcpyHostToDevice, b->stream);
  if (e == hipSuccess) e = gvom::launch_batch_insert(b->dtab, b->grid, b->dstamps, b->stream);
  if (e == hipSuccess) e = gvom::launch_batch_export(b->dtab, b->grid, b->dstamps, b->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(b->hstamps, b->dstamps, gvom::kStampQueue * sizeof(unsigned long long),
                       hipMemcpyDeviceToHost, b->stream);
  return e;
}

void batch_fail(map_batch_t* b, hipError_t e = hipSuccess) {
  if (getenv("GVOM_DEBUG")) fprintf(stderr, "gvom batch: %s\n", hipGetErrorString(e));
  (void)hipGetLastError();
  for (int i = 0; i < b->k; i++) b->maps[i]->sticky = MAP_E_DEVICE;
}

void drop_graph(map_batch_t* b) {
  if (!b->captured) return;
  (void)hipGraphExecDestroy(b->exec);
  (void)hipGraphDestroy(b->graph);
  b->captured = false;
}

// Fills the step table; the caller has checked every request.
int32_t batch_prepare(map_batch_t* b, const float* const* xyz_dev, const int64_t* n,
                      const float* poses, const uint32_t* flags, const map_2d_t* out2d,
                      int32_t* const* lut_dev, map_voxel_t* const* data_dev, const int64_t* cap,
                      int64_t* const* n_occupied_dev, const int32_t (*S)[3]) {
  gvom::BatchTables* t = b->htab;
  gvom::BatchStep& st = t->st;
  st.nmaps = b->k;
  st.pre_rays[0] = st.pre_trace[0] = st.pre_col[0] = st.pre_surf[0] = 0;
  st.pre_lwrite[0] = 0;
  int64_t t64 = 0;
  int64_t all = 0;  // points
  size_t surf_lds = 0;
  for (int i = 0; i < b->k; i++) {
    t64 += tiles64(b->maps[i]);
    all += n[i];
  }
  // (see kBatchTracePoints; the grid is what the device holds)
  const int64_t fill = all / (b->grid.trace / 2);
  const int64_t points = fill < 1 ? 1 : std::min<int64_t>(fill, gvom::kBatchTracePoints);
  for (int i = 0; i < b->k; i++) {
    map_t* m = b->maps[i];
    bool full = false;
    const int32_t s = prepare_insert(m, xyz_dev[i], n[i], poses + 12 * i, flags[i], S[i],
                                     &t->ins[i], &t->clr[i], &full, m->seg_len);
    if (s) return s;  // allocation failure
    // blocks take `points` points' rays each, from a queue (see k_b_trace)
    const int64_t tb = (n[i] + points - 1) / points;
    if (tb < t->ins[i].trace_blocks) {
      m->last_trace_blocks -= t->ins[i].trace_blocks - tb;
      t->ins[i].trace_blocks = (int32_t)tb;
    }
    const bool lut = lut_dev && lut_dev[i];
    column_args(m, &out2d[i], lut, &t->col[i]);
    m->ranked = false;
    m->empty = false;
    m->version = gvom::next_version();
    surface_args(m, &out2d[i], lut, &t->sur[i]);
    if (lut) {
      lut_args(m, lut_dev[i], data_dev ? data_dev[i] : nullptr, cap ? cap[i] : 0,
               n_occupied_dev[i], &t->lut[i]);
      t->lut[i].scanned = t->lut[i].nsuper > gvom::kWaveSupers;
    }
    const int64_t C = (int64_t)m->p.nx * m->p.ny;
    const int ray_blocks = (int)((n[i] + gvom::kRayBlock - 1) / gvom::kRayBlock);
    st.surf_H[i] = surf_halo(m);
    const int tile = surf_tile(m, t64);
    st.surf_tile[i] = tile;
    const size_t lds = gvom::surface_lds(st.surf_H[i], tile);
    surf_lds = lds > surf_lds ? lds : surf_lds;
    const int tiles_y = (m->p.ny + tile - 1) / tile;
    const int tiles = ((m->p.nx + tile - 1) / tile) * tiles_y;
    const int lw_by = (m->d.nby + 3) / 4;
    const int lw = ((m->p.nx + 3) / 4) * lw_by;
    st.ray_blocks[i] = n[i] > 0 ? ray_blocks : 0;
    st.pre_rays[i + 1] = st.pre_rays[i] + st.ray_blocks[i] + gvom::clear_blocks(t->clr[i]);
    st.pre_trace[i + 1] = st.pre_trace[i] + t->ins[i].trace_blocks;
    st.pre_col[i + 1] = st.pre_col[i] + (int)((C + 255) / 256);
    st.pre_surf[i + 1] = st.pre_surf[i] + tiles;
    st.pre_lwrite[i + 1] = st.pre_lwrite[i] + (lut ? lw : 0);
    st.surf_tiles_y[i] = tiles_y;
    st.lw_by[i] = lw_by;
    st.nz_magic[i] = gvom::nz_magic(m->p.nz);
    st.last_is_lut[i] = lut ? 1 : 0;
    (void)full;  // a whole-window clear is the plan's single full box
  }
  // the recorded launches hold the surface pass's LDS: once it changes (a tile was
  // set), they are recorded anew
  if (surf_lds != b->grid.surf_lds) {
    drop_graph(b);
    b->grid.surf_lds = surf_lds;
  }
  return MAP_OK;
}

int32_t batch_run(map_batch_t* b) {
  hipError_t e = hipSuccess;
  if (b->use_graph) {
    if (!b->captured) {
      e = hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal);
      if (e == hipSuccess) {
        const hipError_t e1 = enqueue_batch(b);
        e = hipStreamEndCapture(b->stream, &b->graph);
        if (e == hipSuccess) e = e1;
      }
      if (e == hipSuccess) e = hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0);
      if (e != hipSuccess) {
        batch_fail(b, e);
        return MAP_E_DEVICE;
      }
      b->captured = true;
    }
    e = hipGraphLaunch(b->exec, b->stream);
  } else {
    e = enqueue_batch(b);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
  if (e != hipSuccess) {
    batch_fail(b, e);
    return MAP_E_DEVICE;
  }
  for (int i = 0; i < b->k; i++) {
    unsigned long long end = 0;
    for (int t = 0; t < gvom::kStampSlots; t++)
      end = std::max(end, b->hstamps[gvom::kStampEnds + t * gvom::kMaxBatch + i]);
    b->last_ms[i] = (double)(end - b->hstamps[0]) / b->clock_khz;
  }
  return MAP_OK;
}

int32_t batch_check(map_batch_t* b, const float* const* xyz_dev, const int64_t* n,
                    const float* poses, const uint32_t* flags, const map_2d_t* out2d,
                    int32_t* const* lut_dev, const int64_t* cap, int64_t* const* n_occupied_dev,
                    int32_t (*S)[3]) {
  if (!b || !xyz_dev || !n || !poses || !flags || !out2d) return MAP_E_INVALID;
  for (int i = 0; i < b->k; i++) {
    if (flags[i] & MAP_STATS_DISTINCT) return MAP_E_INVALID;
    if (!valid_2d(&out2d[i])) return MAP_E_INVALID;
    if (lut_dev && lut_dev[i] && (!n_occupied_dev || !n_occupied_dev[i] || (cap && cap[i] < 0)))
      return MAP_E_INVALID;
    const int32_t s = check_insert(b->maps[i], xyz_dev[i], n[i], poses + 12 * i, flags[i], S[i]);
    if (s) return s;
  }
  // work the caller enqueued on the maps' own streams finishes first (each
  // distinct stream is waited for once)
  hipStream_t seen[gvom::kMaxBatch];
  int ns = 0;
  for (int i = 0; i < b->k; i++) {
    const hipStream_t st = b->maps[i]->stream;
    bool dup = false;
    for (int j = 0; j < ns && !dup; j++) dup = seen[j] == st;
    if (dup) continue;
    seen[ns++] = st;
    if (hipStreamSynchronize(st) != hipSuccess) {
      batch_fail(b);
      return MAP_E_DEVICE;
    }
  }
  return MAP_OK;
}

}  // namespace

extern "C" {

int32_t map_batch_create(map_t* const* maps, int32_t k, void* stream, map_batch_t** out) {
  if (!out) return MAP_E_INVALID;
  *out = nullptr;
  if (!maps || k < 1 || k > gvom::kMaxBatch) return MAP_E_INVALID;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return MAP_E_DEVICE;
  for (int i = 0; i < k; i++) {
    if (!maps[i] || maps[i]->device != dev || maps[i]->sticky) return MAP_E_INVALID;
    for (int j = 0; j < i; j++)
      if (maps[j] == maps[i]) return MAP_E_INVALID;
  }
  map_batch_t* b = new (std::nothrow) map_batch_t();
  if (!b) return MAP_E_OOM;
  b->k = k;
  for (int i = 0; i < k; i++) b->maps[i] = maps[i];
  b->stream = (hipStream_t)stream;
  if (!b->stream) {  // graphs cannot be captured on the null stream: use an own stream
    if (hipStreamCreateWithFlags(&b->stream, hipStreamNonBlocking) != hipSuccess) {
      delete b;
      return MAP_E_DEVICE;
    }
    b->own_stream = true;
  }
  b->device = dev;
  b->n_cu = maps[0]->n_cu;
  b->use_graph = true;
  int khz = 0;
  if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0)
    khz = 100000;
  b->clock_khz = khz;
  size_t lut = 0;
  bool scan = false;
  int64_t cols = 0, units = 0;  // virtual blocks of the column and the table pass
  for (int i = 0; i < k; i++) {
    const size_t s = gvom::lut_lds(maps[i]->p.nz);
    lut = s > lut ? s : lut;
    scan |= n_col(maps[i]) > 4096 * (int64_t)gvom::kWaveSupers;
    cols += (n_col(maps[i]) + 255) / 256;
    units += (int64_t)((maps[i]->p.nx + 3) / 4) * ((maps[i]->d.nby + 3) / 4);
  }
  const int cu = b->n_cu;
  // Grids, no larger than the maps' virtual blocks.  The traversal's as many blocks as
  // are resident (with eight per CU, one of them waiting for a place, 922 us instead of
  // 770).  The bandwidth-bound column and table passes 64 per CU: a block that goes on
  // to its next virtual block starts that one's chain of loads only behind the last
  // one's stores, a new block at once (32 maps, with 8 / 16 / 64 / 128 / 512 per CU: table
  // 562 / 546 / 521 / 500 / 473 us, column 63 / 61 / 60 / 61 / 61).
  const auto at_most = [](int64_t a, int64_t c) { return (int)(a < c ? a : c); };
  b->grid = gvom::BatchGrid{cu * 4, cu * gvom::kTraceWavesPerSimd, at_most(cu * 64, cols), cu * 2,
                            at_most(cu * 64, units), k * gvom::box_fold_blocks(),
                            scan ? k : 0, 0, lut};
  hipError_t e = gvom::dev_alloc((void**)&b->dtab, sizeof(gvom::BatchTables));
  if (e == hipSuccess) e = hipHostMalloc((void**)&b->htab, sizeof(gvom::BatchTables), 0);
  if (e == hipSuccess) e = gvom::dev_alloc((void**)&b->dstamps, (gvom::kStampQueue + 1) * 8);
  if (e == hipSuccess) e = hipHostMalloc((void**)&b->hstamps, gvom::kStampQueue * 8, 0);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    map_batch_destroy(b);
    return MAP_E_OOM;
  }
  memset(b->htab, 0, sizeof(gvom::BatchTables));
  *out = b;
  return MAP_OK;
}

int32_t map_batch_destroy(map_batch_t* b) {
  if (!b) return MAP_OK;
  (void)hipStreamSynchronize(b->stream);
  drop_graph(b);
  (void)gvom::dev_free(b->dtab);
  (void)hipHostFree(b->htab);
  (void)gvom::dev_free(b->dstamps);
  (void)hipHostFree(b->hstamps);
  if (b->own_stream) (void)hipStreamDestroy(b->stream);
  delete b;
  return MAP_OK;
}

int32_t map_batch_set_graph(map_batch_t* b, int32_t enable) {
  if (!b) return MAP_E_INVALID;
  b->use_graph = enable != 0;
  return MAP_OK;
}

int32_t map_batch_step(map_batch_t* b, const float* const* xyz_dev, const int64_t* n,
                       const float* poses, const uint32_t* flags, const map_2d_t* out2d,
                       int32_t* const* lut_dev, map_voxel_t* const* data_dev,
                       const int64_t* cap, int64_t* const* n_occupied_dev) {
  int32_t S[gvom::kMaxBatch][3];
  int32_t s = batch_check(b, xyz_dev, n, poses, flags, out2d, lut_dev, cap, n_occupied_dev, S);
  if (s) return s;
  s = batch_prepare(b, xyz_dev, n, poses, flags, out2d, lut_dev, data_dev, cap, n_occupied_dev, S);
  if (s) return s;
  return batch_run(b);
}

int32_t map_batch_latency(const map_batch_t* b, double* ms) {
  if (!b || !ms) return MAP_E_INVALID;
  for (int i = 0; i < b->k; i++) ms[i] = b->last_ms[i];
  return MAP_OK;
}

int32_t map_batch_autotune(map_batch_t* b, const float* const* xyz_dev, const int64_t* n,
                           const float* poses, const uint32_t* flags, const map_2d_t* out2d,
                           const char* cache_path, map_tuning_t* chosen) {
  if (!b) return MAP_E_INVALID;
  int32_t S[gvom::kMaxBatch][3];
  int32_t s = batch_check(b, xyz_dev, n, poses, flags, out2d, nullptr, nullptr, nullptr, S);
  if (s) return s;
  // cache key: device, compute units, map shapes, point-count range
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, b->device) != hipSuccess) return MAP_E_DEVICE;
  int64_t ntot = 0;
  for (int i = 0; i < b->k; i++) ntot += n[i];
  int bucket = 0;
  for (int64_t v = ntot / b->k; v > 1; v >>= 1) bucket++;
  std::string key = std::string(prop.gcnArchName) + "/cu" + std::to_string(b->n_cu) + "/n2^" +
                    std::to_string(bucket);
  for (int i = 0; i < b->k; i++) {
    const map_t* m = b->maps[i];
    key += "/" + std::to_string(m->p.nx) + "x" + std::to_string(m->p.ny) + "x" +
           std::to_string(m->p.nz);
  }
  for (char& c : key)
    if (c == ' ') c = '_';
  // a surface tile of 32 stands for the library's choice (32, in a large launch 64)
  const auto apply = [&](const map_tuning_t& t) {
    for (int i = 0; i < b->k; i++)
      if (map_set_tuning(b->maps[i], &t) == MAP_OK && t.surface_tile == 32)
        b->maps[i]->tile_auto = true;
  };
  map_tuning_t best{0, 0, 0};
  bool cached = false;
  if (cache_path) {
    if (FILE* f = fopen(cache_path, "r")) {
      char line[8192];
      while (fgets(line, sizeof(line), f)) {
        char k2[8000];
        int a = 0, w = 0, tl = 0;
        if (sscanf(line, "%7999s %d %d %d", k2, &a, &w, &tl) == 4 && key == k2) {
          best.seg_len = a;
          best.trace_waves_per_cu = w;
          best.surface_tile = tl;
          cached = true;
        }
      }
      fclose(f);
    }
  }
  if (!cached) {
    // segment length x traversal waves per CU x surface tile
    const int segs[3] = {6, 8, 16}, wpcs[2] = {16, 28}, tiles[2] = {16, 32};
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return MAP_E_DEVICE;
    float best_ms = 1e30f;
    for (int si = 0; si < 3; si++)
      for (int wi = 0; wi < 2; wi++)
        for (int ti = 0; ti < 2; ti++) {
        const map_tuning_t t{segs[si], wpcs[wi], tiles[ti]};
        apply(t);
        float tot = 0.0f;
        for (int rep = 0; rep < 3; rep++) {
          for (int i = 0; i < b->k; i++) map_reset(b->maps[i]);
          s = batch_check(b, xyz_dev, n, poses, flags, out2d, nullptr, nullptr, nullptr, S);
          if (!s) s = batch_prepare(b, xyz_dev, n, poses, flags, out2d, nullptr, nullptr, nullptr,
                                    nullptr, S);
          if (s) return s;
          (void)hipEventRecord(e0, b->stream);
          s = batch_run(b);
          (void)hipEventRecord(e1, b->stream);
          (void)hipEventSynchronize(e1);
          if (s) return s;
          float ms = 0.0f;
          (void)hipEventElapsedTime(&ms, e0, e1);
          if (rep > 0) tot += ms;  // the first run of a setting warms it up
        }
        if (tot < best_ms) {
          best_ms = tot;
          best = t;
        }
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (cache_path) {
      if (FILE* f = fopen(cache_path, "a")) {
        fprintf(f, "%s %d %d %d\n", key.c_str(), best.seg_len, best.trace_waves_per_cu,
                best.surface_tile);
        fclose(f);
      }
    }
  }
  apply(best);
  for (int i = 0; i < b->k; i++) map_reset(b->maps[i]);
  if (chosen) *chosen = best;
  return MAP_OK;
}

const char* map_status_str(int32_t s) {
  switch (s) {
    case MAP_OK: return "ok";
    case MAP_E_INVALID: return "invalid argument";
    case MAP_E_POSE: return "non-finite pose";
    case MAP_E_SENSOR_OUTSIDE: return "sensor outside the map window";
    case MAP_E_RANGE: return "sensor position out of range";
    case MAP_E_CAPACITY: return "output buffer too small";
    case MAP_E_OOM: return "device allocation failed";
    case MAP_E_DEVICE: return "HIP runtime error";
    default: return "unknown status";
  }
}

}  // extern "C"
