// Internal declarations shared by the host code and the kernels of libgvom.
//
// Storage layout on the device (per map):
//   hits, passes, min_qz : int32 per voxel, TOROIDAL: world voxel g is stored
//                          at storage coordinate s = (g mod nx, g mod ny,
//                          g mod nz), so a moving window only clears the slabs
//                          it enters.  Columns are grouped in 4 x 4 bricks:
//                          voxel s lives at col_base(sx, sy) + 16 sz, so one
//                          64-byte line holds one z level of a brick and
//                          neighbouring columns share lines.
//   occ                  : uint64[nx*ny][W], W = ceil(nz/64): bit (s mod 64) of
//                          word s/64 is set iff storage z = s of that column
//                          holds a return (hits >= 1).
// "ro" is the ring offset origin mod n per axis: window-local coordinate l
// is stored at (l + ro) mod n.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gvom.h"

namespace gvom {

// Device allocations of the library go through these two calls, which keep
// the process-wide total that map_set_device_memory_limit caps.
hipError_t dev_alloc(void** p, size_t bytes);
hipError_t dev_free(void* p);

struct Dims {
  int32_t nx, ny, nz, W;  // W = occupancy words per column
  int32_t ro[3];          // ring offsets
  int32_t nby;            // bricks along y = ceil(ny / 4)
  int64_t vs;             // storage voxels = ceil(nx/4) * nby * nz * 16
};

// Storage index of z = 0 of storage column (sx, sy); z adds 16 per level.
__host__ __device__ __forceinline__ int32_t col_base(const Dims& d, int32_t sx, int32_t sy) {
  return ((((sx >> 2) * d.nby + (sy >> 2)) * d.nz) << 4) + ((sy & 3) << 2) + (sx & 3);
}

constexpr int kStripes = 16;  // independent segment counters of the ray pass
static_assert(kStripes == 16, "the traversal scans the stripes in one row of lanes");

// Sensor box of the segmented traversal: every ray starts in the sensor's
// voxel, so the cells around it take the passes of thousands of waves and
// device atomics on their few cache lines serialize.  Passes of cells inside a
// kBoxXY x kBoxXY x kBoxZ box around the sensor are summed per block in LDS,
// flushed into one of kBoxReps replicas of the box, and the replicas are
// added into the map by a small fold kernel.
constexpr int kBoxXY = 17;
constexpr int kBoxZ = 9;
constexpr int kBoxCells = kBoxXY * kBoxXY * kBoxZ;
constexpr int kBoxReps = 128;

struct InsertArgs {
  const float* xyz;
  int32_t n;
  int32_t fw;             // firing width (1 = identity order)
  int32_t azimuths;       // n / fw
  float R[9], t[3];
  float inv_r;
  int32_t S[3];           // sensor, Q units
  int32_t O[3];           // window origin, world voxel
  Dims d;
  int32_t* hits;
  int32_t* passes;
  int32_t* minqz;
  unsigned long long* occ;
  unsigned long long* stats;   // [8 global counters][kStripes segment counters]
  uint32_t* touch;             // distinct-voxel bitmaps [2][V/32] or null
  unsigned long long* part_rays;   // per ray block: nonfinite, range, hits, 0
  unsigned long long* part_trace;  // per trace block: passes, distinct passes, updates,
                                   // distinct hits
  int4* rays;                  // per ray (ray-pass lane): {Qx, Qy, Qz, 4 segments + dominant axis}
  int2* witems;                // wave items {ray wave, segment index}, per stripe
  int64_t block_items;         // wave items one ray block has room for
  int32_t seg_len;             // dominant-axis voxels per segment
  int32_t trace_blocks;        // (virtual) blocks of the traversal, kTraceBlock threads each
  // sensor box (segmented traversal): storage coordinate of its first cell
  // and extent per axis; cell (dx, dy, dz) has box index
  // (dx * kBoxXY + dy) * kBoxZ + dz
  int32_t box_s[3];
  int32_t box_e[3];
  int32_t box_far;             // most voxels along an axis from the sensor to a box cell
  int32_t* box_rep;            // [kBoxReps][kBoxCells], zero between inserts
};

constexpr int kBlock = 256;       // threads per block of the plain kernels
constexpr int kRayBlock = 512;    // threads per block of the ray pass (rays regrouped per block)
// threads per block of the traversal (single map and batch): four waves
// share one LDS copy of the sensor box; seven of them fit a CU (72 registers a
// thread, for which one value goes to scratch, in the batch's kernel four; with 64
// registers eight fit, but nine go: 43.1 -> 43.8 us at 131,072 points, 16.0 -> 18.4 at
// 28,800)
constexpr int kTraceBlock = 256;
constexpr int kTraceWavesPerSimd = 7;
// Points per traversal block of a batch, at most: 32 maps of 20,000-330,000 points take 725 us
// with 64, 654 with 128, 648 with 256, 688 with 384 (a block's set-up and flush take as
// long as about 60 points' rays; large blocks leave waves idle at the end).  A step of few
// points takes fewer, so that its blocks take at least every second place on the device:
// one map of 512 x 512 x 64 with 3,000 points, the whole step with 256 points a block
// 351 us, with a block for every eighth / fourth / second / each place 125 / 130 / 133 /
// 132; of 1024 x 1024 x 16 with 60,000 points 586, 585 / 498 / 487 / 473.
constexpr int kBatchTracePoints = 256;

// Blocks of the sensor-box fold that follows the segmented traversal.
int box_fold_blocks();

// Segments one ray can produce at most.
int64_t max_segments(const Dims& d, int32_t seg_len);

struct ColumnArgs {
  Dims d;
  const int32_t* hits;
  const int32_t* passes;
  const int32_t* minqz;
  const unsigned long long* occ;
  double res;
  int32_t n_lo, n_hi;
  int32_t dens_num, dens_den;
  float* height;
  float* density;
  uint8_t* flags;
  int32_t* hq;            // ground height Q per local pixel, INT32_MIN = undefined
  unsigned long long* defbits;  // bit c % 64 of word c / 64: pixel c has a height
  int32_t* colpre;        // null, or the table export's counting pass (see LutArgs)
  int32_t* group_cnt;
};

struct SurfaceArgs {
  int32_t nx, ny;
  const int32_t* hq;
  const uint32_t* defbits;  // the column pass's bits, as 32-bit words
  const int32_t* imported;  // kWild set: heights may lie outside the window
  int32_t half_fit;
  int32_t search_d;
  int64_t tau_q;
  double q2m;             // metres per Q unit = res / 65536
  float* slope;
  float* rough;
  uint8_t* flags;
  // the table export's group counts (see LutArgs), turned into prefixes and sums
  // of super groups by this launch; rank_n = groups, 0: none
  int32_t* rank_cnt;
  int32_t rank_n;
  int32_t* rank_sum;
};

// Super groups of ranks whose sums every region of a table export scans by itself, one a
// lane; more of them are scanned once before (k_lut_scan, k_b_lut_scan), since every
// further 64 cost each region a round.  Export after a 2D export, scanned in regions /
// before: 512 x 512 x 64 (64 super groups) 31.3 / 33.8 us, 640 x 640 x 64 (100) 46.0 /
// 45.4, 1024 x 1024 x 16 (256) 43.8 / 38.1, 1024 x 1024 x 96 191.9 / 184.5; a batched
// step of 32 maps of 1024 x 1024 x 16 4394 / 3948.
constexpr int kWaveSupers = 64;

// What an import found: content it refuses; a lowest return outside its voxel, which
// the map then holds until it is emptied or combined anew.
constexpr int32_t kBadContent = 1, kWild = 2;

struct LutArgs {
  Dims d;
  const int32_t* hits;
  const int32_t* passes;
  const int32_t* minqz;
  const unsigned long long* occ;
  int32_t* lut;
  map_voxel_t* data;
  int64_t cap;
  // a column's first rank = the sums of the super groups before its own + its
  // group's prefix within that + its rank within its group
  int32_t* group_cnt;     // per group of 64 window-local columns: its prefix within its
                          // super group
  int32_t* super_sum;     // per super group of 64 groups: their sum, or the exclusive
                          // prefix of the sums (scanned != 0)
  int32_t* colpre;        // per window-local column: exclusive rank within its group
  int32_t nsuper, scanned;
  int64_t* n_occupied;
};

struct DensityArgs {
  Dims d;
  const int32_t* hits;
  const int32_t* passes;
  const unsigned long long* occ;
  float* out;             // [nx*ny*nz], window-local table order
};

// Per-column features of the gap-fill surrogate ([nx][ny][16]; undefined values
// are 0):
//  0 sum of hits, 1 sum of passes, 2 occupied voxels, 3 occupied fraction,
//  4 ground height, 5 height of the highest occupied voxel, 6 mean of the
//  occupied voxels' lowest returns, 7 height defined, 8 density of the ground
//  voxel, 9 obstacle-band density, 10 slope, 11 roughness, 12 slope defined,
//  13 horizontal distance of the column centre to the sensor, 14 sensor height
//  above the ground, 15 column thinned.  A thinned column keeps only 13, 15.
struct FeatArgs {
  Dims d;
  const int32_t* hits;
  const int32_t* passes;
  const int32_t* minqz;
  const unsigned long long* occ;
  int32_t O[3];
  double res;
  double sx, sy, sz;  // sensor position, m
  const float* height;
  const float* density;
  const float* slope;
  const float* rough;
  const uint8_t* flags;
  const uint8_t* thin;  // may be null
  float* feat;
};

struct CostArgs {
  int64_t n;              // pixels
  const float* slope;
  const float* rough;
  const float* density;
  const uint8_t* flags;
  float w[8];             // slope, rough, density, positive, hard, soft, negative, unknown
  float* cost;
};

// The slabs a moved window takes over (storage coordinates, cut where they
// wrap), and which of every column's levels stay.
constexpr int kClearBoxes = 6;
struct ClearArgs {
  Dims d;
  int32_t* hits;
  int32_t* passes;
  int32_t* minqz;
  unsigned long long* occ;
  int32_t nbox;                        // 0: nothing to clear
  int32_t box[kClearBoxes][6];         // [x0, x1) x [y0, y1) x [z0, z1)
  int32_t pre[kClearBoxes + 1];        // words (16 bytes of passes) of the boxes before
  int32_t nslab;                       // the boxes that span every level come first
  unsigned long long keep[2];          // occupancy bits outside the z boxes
};

// ---- batches of maps ------------------------------------------------------
constexpr int kMaxBatch = 64;

// Clock values of a step, in device memory (64-bit words): its start, then kStampSlots
// x kMaxBatch completion maxima of the maps, then the traversal's queue.  A map's blocks
// spread over its slots, which lie in lines of their own: an atomic on one address costs
// 46 ns behind the last one, so with one word per map the 16,384 blocks of the table pass
// of four maps of 1024 x 1024 x 16 took 756 us, with the slots 127.
constexpr int kStampSlots = 16;
constexpr int kStampEnds = 8;  // (the start has a line of its own)
constexpr int kStampQueue = kStampEnds + kStampSlots * kMaxBatch;

// Per-step table of a batch: virtual-block prefixes of every stage (block b of
// stage S belongs to the map m with pre[m] <= b < pre[m+1]) and per-map
// launch constants.  Lives in device memory, uploaded once per step.
struct BatchStep {
  int32_t nmaps;
  int32_t pre_rays[kMaxBatch + 1];   // ray blocks and, after them, clear blocks
  int32_t ray_blocks[kMaxBatch];
  int32_t pre_trace[kMaxBatch + 1];
  int32_t pre_col[kMaxBatch + 1];
  int32_t pre_surf[kMaxBatch + 1];
  int32_t pre_lwrite[kMaxBatch + 1];
  int32_t surf_tile[kMaxBatch];    // 16, 32 or 64
  int32_t surf_tiles_y[kMaxBatch];
  int32_t surf_H[kMaxBatch];
  int32_t lw_by[kMaxBatch];
  uint32_t nz_magic[kMaxBatch];
  int32_t last_is_lut[kMaxBatch];
};

struct BatchTables {
  BatchStep st;
  ClearArgs clr[kMaxBatch];
  InsertArgs ins[kMaxBatch];
  ColumnArgs col[kMaxBatch];
  SurfaceArgs sur[kMaxBatch];
  LutArgs lut[kMaxBatch];
};

struct BatchGrid {
  int rays, trace, col, surf, lwrite;  // persistent grid sizes
  int fold;                                                   // maps x sensor-box fold blocks
  int scan;                            // maps, if one has more than kWaveSupers super groups
  size_t surf_lds, lut_lds;
};

// Enqueues one batched step (all stages of all maps) reading `tab` (device).
// stamps: see kStampSlots (wall clock:
// the latest end of its last-stage blocks).
hipError_t launch_batch_insert(const BatchTables* tab, const BatchGrid& g,
                               unsigned long long* stamps, hipStream_t s);
hipError_t launch_batch_export(const BatchTables* tab, const BatchGrid& g,
                               unsigned long long* stamps, hipStream_t s);
size_t surface_lds(int H, int tile);
// The library's choice of the surface pass's tile edge; tiles64 = tiles of 64
// pixels in the launch.
int surface_tile_for(int H, int64_t tiles64, int n_cu);
size_t lut_lds(int nz);
uint32_t nz_magic(int nz);

// Launchers (all enqueue on `s`, return the launch status).
hipError_t launch_clear(const ClearArgs& a, hipStream_t s);
// The ray pass and, beside it, the clears of the moved window (which nothing in
// it touches).
hipError_t launch_rays(const InsertArgs& a, const ClearArgs& c, hipStream_t s);
// Blocks of kRayBlock threads that clear c's boxes.
int clear_blocks(const ClearArgs& c);
hipError_t launch_trace(const InsertArgs& a, bool distinct, hipStream_t s);
hipError_t launch_column(const ColumnArgs& a, hipStream_t s);
hipError_t launch_surface(const SurfaceArgs& a, int tile, hipStream_t s);  // tile 16, 32 or 64
// ranked: colpre, group_cnt and super_sum already hold this state's ranks;
// otherwise they are made first
hipError_t launch_lut(const LutArgs& a, bool ranked, hipStream_t s);
hipError_t launch_import(const Dims& d, const int32_t* lut, const map_voxel_t* data,
                         int64_t n_data, int32_t* hits, int32_t* passes, int32_t* minqz,
                         unsigned long long* occ, int32_t origin_z, int32_t* err,
                         hipStream_t s);
hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
// out[0..3] = column sums of the ray pass's per-block counters parts[nblocks][4].
hipError_t launch_sum_ray_parts(const unsigned long long* parts, int64_t nblocks,
                                unsigned long long* out, hipStream_t s);
hipError_t launch_density(const DensityArgs& a, hipStream_t s);
hipError_t launch_features(const FeatArgs& a, hipStream_t s);
// Empties the window-local columns marked in `thin` (null: all of them) of a
// map whose occupancy words agree with its voxels.
hipError_t launch_thin(const Dims& d, const uint8_t* thin, int32_t* hits, int32_t* passes,
                       int32_t* minqz, unsigned long long* occ, hipStream_t s);
hipError_t launch_costmap(const CostArgs& a, hipStream_t s);
// Exclusive prefix of base[0..nb) in place (one block); *total = the sum.
hipError_t launch_scan_i32(int32_t* base, int nb, int64_t* total, hipStream_t s);

}  // namespace gvom
