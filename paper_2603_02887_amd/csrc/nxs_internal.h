// Internal declarations shared by the HIP translation units of libnxs.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nxs.h"

namespace nxs {

// Per-view parameters, one entry per view in a device table.
struct ViewDev {
  float R[9];
  float t[3];
  float fx, fy, cx, cy, znear;
  float campos[3];          // camera centre in world space, -R^T t
  int32_t width, height;
  int32_t tiles_x, tiles_y;
  int32_t tile_off;         // first global tile of this view
  int32_t cell_off;         // first cell (block of tiles, bin.hip) of this view
  int32_t cells_x;          // cells per row
  int32_t pad_;
  int64_t pix_off;          // first pixel of this view in per-pixel state buffers
  float* rgb;               // [H, W, 3]
  float* trans;             // [H, W]
  int32_t* od;              // [H, W] or null
  const float* g_rgb;       // backward: dLoss/drgb [H, W, 3]
  const float* g_trans;     // backward: dLoss/dtrans [H, W] or null
};

struct GaussDev {
  const float* means;
  const float* scales;
  const float* quats;
  const float* opac;
  const float* sh;
  int32_t n;
  int32_t sh_degree;
};

// Per projected slot (slot = view * n + gaussian) arrays written by the projection.
struct ProjDev {
  uint32_t* depth_key;      // float32 depth bits; 0xFFFFFFFF when culled
  // rectangle (x0 | x1 << 16, y0 | y1 << 16) in blocks of 8x8 pixels, all ones
  // when culled (the tiles it covers are tile_rect() of it); `small`: as
  // small_rect() words
  uint2* trect;
  bool small;
  // 3 float4 per slot:
  //   (u_hi, u_lo, v_hi, v_lo)  image-plane centre as float hi + lo parts
  //   (A', B', C', log2 aleph)  log2(alpha) = log2 aleph + A' dx^2 + B' dx dy + C' dy^2
  //   (r, g, b, 0)              emission
  float4* rec;
};

// Device counters filled by the projection: total instances, depth-bit range.
struct Counters {
  unsigned long long total;
  uint32_t dmin, dmax;
  // the depth sort's digits (shift | width << 8 | kPassActive per pass),
  // from dmin ^ dmax
  uint32_t plan[4];
  // a deferred render that cannot complete (kFail* bits; 0 otherwise): the
  // kernels after the emission then do nothing
  uint32_t fail;
  uint32_t pad_;
};
constexpr uint32_t kFailCapacity = 1u;   // more instances than the capacity
constexpr uint32_t kFailPlan = 2u;       // the depth sort skipped a pass it needs

// The outcome of the deferred renders on a context since the host last read
// it (device memory, cleared by the host).
struct DeferredStatus {
  unsigned long long need;   // largest instance count a failed render needed
  unsigned long long last;   // instance count of the latest deferred render
  uint32_t fail;             // OR of their kFail* bits
  uint32_t count;            // failed renders
  uint32_t last_fail;        // kFail* bits of the latest deferred render
  uint32_t pad_;
};

// What the projection's final fold checks for a deferred render, and where
// it also writes its results in pinned host memory (so that no copy command
// follows it).
struct DeferCheck {
  unsigned long long capacity;   // instance capacity (~0: not deferred)
  int first_pass;                // first depth-sort pass launched (0 or 1)
  DeferredStatus* status;        // device status, updated by every deferred render
  DeferredStatus* status_host;   // pinned copy of it after the update, or null
  Counters* counters_host;       // pinned copy of the counters, or null
};

// Inclusive sum over the lanes of a wave (every lane active): within each
// 16-lane row by four DPP row shifts (a lane whose source lies before its
// row adds 0), then the three lower rows' totals, read by readlane.  Integer
// sums: the same result as any other order.
__device__ __forceinline__ uint32_t wave_inclusive_scan_u32(uint32_t x) {
  int v = (int)x;
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
  const int r0 = __builtin_amdgcn_readlane(v, 15);
  const int r1 = __builtin_amdgcn_readlane(v, 31);
  const int r2 = __builtin_amdgcn_readlane(v, 47);
  const int row = (int)(threadIdx.x & 63) >> 4;
  v += (row >= 1 ? r0 : 0) + (row >= 2 ? r1 : 0) + (row >= 3 ? r2 : 0);
  return (uint32_t)v;
}

// A wave's reduction under an associative, commutative op (every lane active):
// within each 16-lane row by four DPP row shifts (a lane whose source lies
// before its row combines the identity), then the four rows' last lanes,
// read by readlane; the result is the same on every lane.
template <typename Op>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t x, uint32_t identity, Op op) {
  const int id = (int)identity;
  uint32_t v = x;
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x111, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x112, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x114, 0xF, 0xF, false));
  v = op(v, (uint32_t)__builtin_amdgcn_update_dpp(id, (int)v, 0x118, 0xF, 0xF, false));
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 15);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 31);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 47);
  const uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
  return op(op(r0, r1), op(r2, r3));
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x) {
  return wave_reduce_u32(x, 0u, [](uint32_t a, uint32_t b) { return a + b; });
}
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
  return wave_reduce_u32(x, 0xFFFFFFFFu, [](uint32_t a, uint32_t b) { return min(a, b); });
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
  return wave_reduce_u32(x, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
}

// For each of ITEMS digits per lane: the lanes of the wave whose digit equals
// this lane's (width bits; lo / hi hold the valid lanes on entry).  Per bit and
// digit one bit extract, one compare whose mask is the ballot, and two
// three-input operations; the digits side by side, so that their chains
// overlap.  (With the mask inverted by selects, eight instructions, and one
// digit after another, a scatter pass over 1M keys took 11.6 us instead of
// 10.8, over 48M keys 323 instead of 286.)
template <int ITEMS>
__device__ __forceinline__ void match_digits(const uint32_t (&d)[ITEMS], int width,
                                             uint32_t (&lo)[ITEMS], uint32_t (&hi)[ITEMS]) {
  for (int b = 0; b < width; ++b) {
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const uint32_t s = (uint32_t)__builtin_amdgcn_sbfe((int)d[r], (uint32_t)b, 1u);
      const uint64_t m = __builtin_amdgcn_ballot_w64(s != 0u);
      lo[r] &= ~((uint32_t)m ^ s);
      hi[r] &= ~((uint32_t)(m >> 32) ^ s);
    }
  }
}

// How many of the lanes in the mask lie below this one.
__device__ __forceinline__ uint32_t lanes_below(uint32_t lo, uint32_t hi) {
  return __builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
}

// A rectangle of 8x8 blocks in tiles of 2^ax x 2^ay blocks (culled: stays so).
__host__ __device__ __forceinline__ uint2 tile_rect(uint2 r, int ax, int ay) {
  if (r.x == 0xFFFFFFFFu) return r;
  r.x = ((r.x & 0xFFFFu) >> ax) | ((r.x >> 16 >> ax) << 16);
  r.y = ((r.y & 0xFFFFu) >> ay) | ((r.y >> 16 >> ay) << 16);
  return r;
}

// A rectangle in one word (x0 | y0 << 8 | x1 << 16 | y1 << 24), where no
// coordinate exceeds 254; all ones when culled.
constexpr int kSmallRectBlocks = 255;
__host__ __device__ __forceinline__ uint32_t small_rect(uint2 r) {
  return r.x == 0xFFFFFFFFu ? 0xFFFFFFFFu : (r.x | (r.y << 8));
}
__host__ __device__ __forceinline__ uint2 wide_rect(uint32_t w) {
  const bool culled = w == 0xFFFFFFFFu;
  uint2 r;
  r.x = culled ? w : w & 0x00FF00FFu;
  r.y = culled ? w : (w >> 8) & 0x00FF00FFu;
  return r;
}
// rectangle i of an array of either kind
template <bool SMALL>
__device__ __forceinline__ uint2 load_rect(const uint2* rects, int64_t i) {
  if (SMALL) return wide_rect(reinterpret_cast<const uint32_t*>(rects)[i]);
  return rects[i];
}

// The tiles a slot's rectangle covers (0 for a culled slot).
__device__ __forceinline__ uint32_t rect_tile_count(uint2 r) {
  if (r.x == 0xFFFFFFFFu) return 0u;
  return ((r.x >> 16) - (r.x & 0xFFFFu) + 1u) * ((r.y >> 16) - (r.y & 0xFFFFu) + 1u);
}

// The instance count a kernel after the emission works on: 0 for a failed
// deferred render.
__device__ __forceinline__ int64_t live_count(const Counters* c) {
  return c->fail ? 0 : (int64_t)c->total;
}

// Up to this many views travel to the projection as a kernel argument (the
// projection then writes the device view table the later kernels read), so
// that a render needs no host-to-device copy.
constexpr int kArgViews = 8;
struct ViewArgs {
  ViewDev v[kArgViews];
};

// ---- launchers (all enqueue on `s`) ------------------------------------------
// `partials` needs project_partials_size(n) entries.  Also sets `counters`
// (total instances, depth-bit range, depth-sort plan, fail bits from `check`)
// and zeroes clear[0, n_clear).  host_views: null, or the n_views <=
// kArgViews views (host memory, read during the call), which the projection
// writes to `views`; otherwise `views` must already hold them.  Returns
// false if host_views was given but cannot be used (no Gaussians): the
// caller then copies the table itself.  The rectangles are in units of
// 2^unit_x x 2^unit_y pixels, a tile 2^ax x 2^ay units.
size_t project_partials_size(int n);
bool launch_project(const GaussDev& g, ViewDev* views, const ViewDev* host_views, int n_views,
                    float kappa2, float alpha_min, int unit_x, int unit_y, int ax, int ay,
                    const ProjDev& out, uint4* partials, Counters* counters,
                    const DeferCheck& check, uint32_t* clear, int64_t n_clear,
                    hipStream_t s);

constexpr int kPlanPasses = 4;
constexpr int kMaxDigitBits = 9;
constexpr uint32_t kPassActive = 1u << 16;

// Stable LSD radix sort of (u32 key, u32 value) pairs (reduce-then-scan,
// digits of up to kMaxDigitBits): sorts (keys_in, vals_in) by the low nbits
// of the keys (at least one pass), ping-ponging through (k0, v0) and (k1, v1);
// returns which pair holds the result (0 or 1).  vals_in == nullptr: values
// are the input positions.  `counts` needs radix_counts_words(n) u32.
// With `dn`, the number of pairs is read on the device (live_count(dn)) and
// n is only its upper bound, which sizes the counts layout; the grids are
// planned for n_plan pairs (0: n) and their work-groups loop over the chunks
// of a larger count.
size_t radix_counts_words(int64_t n, int parts = 1);
int radix_sort(const uint32_t* keys_in, const uint32_t* vals_in, uint32_t* k0, uint32_t* v0,
               uint32_t* k1, uint32_t* v1, int64_t n, int nbits, uint32_t* counts,
               hipStream_t s, const Counters* dn = nullptr, int64_t n_plan = 0);
// The same sort of `parts` consecutive parts of n pairs, each on its own, with
// its digits read from device memory: plan[p] = shift |
// width << 8 | kPassActive for kPlanPasses passes (an active pass of width 0
// copies).  Passes 1..3 are always active, pass 0 only when three digits of
// kMaxDigitBits do not cover the varying bits.  Enough for keys of up to 32
// varying bits.  first_pass = 0 launches all four passes (an inactive pass 0
// does nothing and pass 1 then reads the input); first_pass = 1 launches
// passes 1..3 only, which is right only if the plan leaves pass 0 inactive
// (the caller checks plan[0] once it has read the counters, and sorts again
// with first_pass = 0 otherwise).  The result is in (k1, v1); returns 1.
// The last pass also writes, in sorted order, each value's tile rectangle
// from `trect` (indexed by value; both arrays of small_rect() words if `small`)
// into rect_out, and its tile count (tiles of 2^ax x 2^ay units) into nt_out unless
// that is null.
int radix_sort_planned(const uint32_t* keys_in, const uint32_t* vals_in, uint32_t* k0,
                       uint32_t* v0, uint32_t* k1, uint32_t* v1, int64_t n, int parts,
                       const uint32_t* plan, int first_pass, uint32_t* counts,
                       const uint2* trect, uint32_t* nt_out, uint2* rect_out, bool small, int ax,
                       int ay, hipStream_t s);

// Depth sort of views of n <= kLocalMax slots each, one work-group per view
// (depth.hip), stable: the slots of view v's visible Gaussians and their tile
// rectangles in order, from v * n on, and vis[v] how many there are.
constexpr int kLocalMax = 8192;
void launch_depth_local(const uint32_t* depth_key, const uint2* trect, int32_t n, int n_views,
                        uint32_t* vis, uint32_t* slots_out, uint2* rect_out, bool small,
                        hipStream_t s);

// Binning in two levels (bin.hip): each view's slots, in depth order or in slot
// order (sorted_slots null), are dealt to cells of 2^sx x 2^sy tiles, and each
// cell's list is expanded into its tiles' lists.  The lists hold the slots in
// the order given; `ranges` says where each tile's lies (cell by cell, not in
// the order of the tiles).
constexpr int kViewCells = 512;       // cells of one view the kernels' tables hold
constexpr int kMaxCells = 4096;       // and of all views
constexpr int kMaxBinViews = 64;
constexpr int kMaxCellTiles = 64;     // a pair's tiles are one bit each
constexpr int kMaxCellChunk = 4096;   // slots counted together
constexpr int kMaxFineGrid = 4096;    // work-groups of the per-segment kernels
//
// With `pack` a list entry's four top bits say which of the tile's 8x8 blocks
// (at most 4, row by row) the slot's rectangle covers, below them the slot
// (kPackedSlots at most); without, it is the slot alone.
constexpr uint32_t kPackMask = 0x0FFFFFFFu;
constexpr int64_t kPackedSlots = int64_t(1) << 28;
struct BinPlan {
  int sx, sy;         // log2 of a cell's tiles per row and column
  int ax, ay;         // log2 of a tile's 8x8 blocks per row and column
  bool pack;
  bool small;         // the rectangles are small_rect() words
  uint32_t n_cells;   // 0: the two-level binning does not apply
  int32_t n;          // slots per view
  int n_views;
  int chunk;          // slots per chunk
  uint32_t cpv;       // chunks per view
  uint32_t seg_shift; // log2 of the pairs of a segment
};
struct BinBuffers {
  uint32_t* counts;      // bin_counts_words
  uint32_t* cells;       // bin_cells_words
  uint32_t* pair_slot;   // one entry per pair (at most one pair per instance)
  uint16_t* pair_rect;
  uint32_t* segs;        // bin_seg_words
  uint32_t* list;        // one entry per instance
  uint2* ranges;         // per tile; those without instances are left as they are
};
// The pairs [first, first + n) of segment k of a cell whose pairs are [begin, end):
// by their number, since first + 2^shift, or a position a step beyond the last
// pair, may not fit 32 bits (as many pairs as instances, 2^32 - 2 at most).
struct PairRange {
  uint32_t first, n;
};
__host__ __device__ __forceinline__ PairRange segment_pairs(uint32_t begin, uint32_t end,
                                                            uint32_t k, uint32_t shift) {
  const uint32_t first = begin + (k << shift), left = end - first;
  return {first, left < (1u << shift) ? left : (1u << shift)};
}
BinPlan plan_bins(const int32_t* tiles_x, const int32_t* tiles_y, int n_views, int32_t n,
                  int tile_w, int tile_h);
size_t bin_counts_words(const BinPlan& p);
size_t bin_cells_words(const BinPlan& p);
size_t bin_seg_words(const BinPlan& p, uint64_t max_pairs);
// Pairs per chunk and cell, and their first positions.
// (vis: the slots of each view to take, the first of its part; null: all)
void launch_bin_count(const BinPlan& p, const BinBuffers& b, const uint2* rects,
                      const uint32_t* vis, const ViewDev* views, const Counters* counters,
                      hipStream_t s);
// The pairs into their cells' lists; nothing if the render has more than
// `capacity` instances.
void launch_bin_scatter(const BinPlan& p, const BinBuffers& b, const uint32_t* sorted_slots,
                        const uint2* rects, const uint32_t* vis, const ViewDev* views,
                        uint64_t capacity, const Counters* counters, hipStream_t s);
// The cells' lists into the tiles' (grids for m_plan instances).
void launch_bin_tiles(const BinPlan& p, const BinBuffers& b, uint64_t m_plan,
                      const ViewDev* views, const Counters* counters, hipStream_t s);

// Renders the two-level binning does not apply to emit every instance and sort
// them all by tile instead (the list entries are the same, pack_mask 0 or
// ~kPackMask; tiles are 2^ax x 2^ay of the rectangles' blocks):
// exclusive scan of ntiles in sorted-slot order and emission of instances.
size_t scan_blocks_size(int64_t n);
// Exclusive scan of the depth-sorted tile counts (nt_sorted), or with
// nt_sorted null of the tile counts of the rectangles in slot order, per block
// of 512 slots (block totals in block_sums; scanned across blocks here
// only when there are more blocks than the emission sums itself).
void launch_emit_scan(const uint32_t* nt_sorted, const uint2* trect, int ax, int ay,
                      int64_t n_slots, uint32_t* scan_local, uint32_t* block_sums, hipStream_t s);
// Writes the instances of the depth-sorted slots (rectangles in
// rect_sorted), or with sorted_slots null of the slots in their own order
// (rectangles in trect); instances at positions >= capacity are not written.
void launch_emit_write(const uint32_t* sorted_slots, const uint2* rect_sorted,
                       const uint2* trect, int ax, int ay, uint32_t pack_mask, int64_t n_slots,
                       int32_t n_gauss, const ViewDev* views, const uint32_t* scan_local,
                       const uint32_t* block_sums, uint32_t capacity, uint32_t* inst_tile,
                       uint32_t* inst_val, hipStream_t s);

// The tile-first order: after a stable sort by tile of instances emitted in
// slot order, each tile's list (ranges) is sorted stably by its slots'
// float32 depth bits (depth_key), in LDS up to kSegMax entries and through
// `temp` (the same positions) beyond; the bits that vary come from the
// projection's counters.  Nothing is done for a failed deferred render.
// (slot_mask: the bits of an entry that are its slot)
constexpr int kSegMax = 4096;
void launch_tile_depth_sort(const uint2* ranges, int64_t n_tiles, const uint32_t* depth_key,
                            const Counters* counters, uint32_t slot_mask, uint32_t* list,
                            uint32_t* temp, hipStream_t s);

// Tile ranges: ranges[tile] = [first, end) of the tile's entries in the
// tile-sorted instance list (tiles without instances keep what the caller
// filled in, normally [0, 0)).
void launch_fill_u32(uint32_t* p, int64_t n, uint32_t value, hipStream_t s);
// m: the number of instances, or with `dn` its upper bound (the count itself
// is then read on the device; the grid is planned for m_plan instances and
// loops beyond them).
void launch_ranges(const uint32_t* inst_tile, int64_t m, uint2* ranges, hipStream_t s,
                   const Counters* dn = nullptr, int64_t m_plan = 0);

struct CompositeParams {
  float log2_alpha_min;
  float t_eps;              // exponential termination threshold (<= 0: never)
  float param;              // operator parameter (c, gamma or v) for models 4..7
  float bg[3];
  int32_t lds_batch;        // list entries gathered per round: 64, 128 or 256
  // list entries: kPackMask (slot, and the blocks it covers above it) or ~0
  uint32_t slot_mask;
};
// pstate: null, or 3 float4 per pixel kept for the backward pass:
//   (L0, L1, L2, T_final), (E_k, tau_k), (U, 0) with E_k the saturating splat's
//   emission (background if none), tau_k the optical depth before it and
//   U = sum_{j<k} E_j alpha_j.
// Composite launch geometry.  schedule: NXS_SCHED_TILES, NXS_SCHED_BLOCKS,
// NXS_SCHED_QUEUE or NXS_SCHED_PERSISTENT (the last two also need `order`
// [2 n_tiles] as scratch and kSchedCounters u32 counters that are zero at
// the launch: kQueues queue counters, then the length-bucket counters; the
// persistent one sizes its grid from the CU count).
struct CompositeLaunch {
  int schedule;
  int tile_w, tile_h;
  int64_t n_tiles;
  const ViewDev* views;
  int n_views;
  const uint2* ranges;
  const uint32_t* inst_val;  // tile-sorted list of projected slots
  const float4* rec;         // the projection's records, per slot
  uint32_t* order;
  uint32_t* sched_counters;
  int n_cu;
};
constexpr int kQueueWavesPerCU = 32;
constexpr int kQueues = 8;   // one per XCD
constexpr int kSchedCounters = 64;
// The tile order the queue schedules consume (longest tile lists first);
// enqueue before launch_composite for NXS_SCHED_QUEUE and NXS_SCHED_PERSISTENT
// (does nothing for the others).
void launch_composite_order(const CompositeLaunch& L, hipStream_t s);
void launch_composite(int model, const CompositeLaunch& L, const CompositeParams& p,
                      float4* pstate, hipStream_t s);

// Path-replay backward of the composite (models 0..4): per-slot moments
// gslot[9 * slot + f], f = sums over the slot's pixels of alpha dLoss/dalpha
// times (1, dx, dy, dx^2, dx dy, dy^2) and of p dLoss/dL (r, g, b),
// accumulated with atomics (the caller zeroes gslot; launch_project_bwd turns
// them into gradients).  `order`: the forward's
// tile order (longest lists first) to walk the tiles in, or null.
void launch_composite_bwd(int model, int tile_w, int tile_h, int64_t n_tiles,
                          const ViewDev* views, int n_views, const uint2* ranges,
                          const uint32_t* inst_val, const float4* rec, const CompositeParams& p,
                          const float4* pstate, float* gslot, const uint32_t* order,
                          hipStream_t s);

// Gradients of the Gaussians' parameters from the per-slot gradients (summed
// over views; overwrites the outputs).
struct GaussGradDev {
  float* means;
  float* scales;
  float* quats;
  float* opac;
  float* sh;
};
// gslot holds each slot's moments from the composite's backward on entry and
// its dL/d(opacity, u, v, A, B, C, r, g, b) on return.
void launch_project_bwd(const GaussDev& g, const ViewDev* views, int n_views,
                        float* gslot, const GaussGradDev& out, hipStream_t s);

// Measured peaks (peaks.hip): `groups` work-groups of independent FP32 FMA
// chains, `iters` steps each (peak_fma_flops of them, out: peak_fma_out_floats
// floats); a float4 copy of n4 elements (n4 < 2^39), one per thread.
int64_t peak_fma_flops(int groups, int iters);
size_t peak_fma_out_floats(int groups);
void launch_peak_fma(float* out, int groups, int iters, hipStream_t s);
void launch_peak_copy(const float4* src, float4* dst, int64_t n4, hipStream_t s);

// Waits for the context's work, then grows its instance buffers to `need`
// instances (api.hip; a pipeline grows every lane to what one of them needed).
nxs_status grow_instance_capacity(nxs_context* ctx, uint64_t need);

}  // namespace nxs
