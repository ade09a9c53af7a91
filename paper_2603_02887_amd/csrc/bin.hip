// Binning in two levels: from the projected slots in depth order (or, tile
// first, in slot order) to each tile's list of slots in that order.
//
// A cell is a block of 2^sx x 2^sy tiles (at most 64).  A slot's rectangle
// covers few cells however many tiles it covers, so the slots are first dealt
// to the cells, and each cell's short list of (slot, rectangle within the
// cell) is then expanded into its tiles' lists:
//
//   cell_count    per chunk of slots and cell: the slots that cover it, and the
//                 tile instances they have in it
//   cell_scan     per cell over the chunks: first positions, totals
//   cell_starts   over the cells: where the pairs, segments and instances begin
//   cell_scatter  the chunk's (slot, cell) pairs, enumerated in order, ranked
//                 stably by cell (wave ballots) and written to the cells' lists
//   seg_count     per segment of a cell's list: instances per tile
//   cell_tiles    per cell: first list position of every (segment, tile), and
//                 the tile ranges
//   seg_emit      64 pairs at a time: each tile takes, by one ballot over the
//                 pairs' blocks in it, the slots that cover it, and writes them
//                 as one run at its position, each with the 8x8 blocks of the
//                 tile it covers (the composite's waves fetch by them)
//
// Every instance is written once, as the 4-byte slot of its list entry, and
// never sorted: the pairs that are moved by cell number one to three per slot.
// Emitting every instance and sorting all of them by tile (two radix passes of
// 8-byte pairs, then the ranges) moved each one five times: 845 us for the 62M
// instances of eight 720p views of 500k Gaussians, 257 us here; 78 against
// 60 us for the 2.69M of the 1080p frame of 1M; 1,650 against 1,150 us for the
// 99M of sixteen views of 3M.
// Every kernel is bound by the latency of its steps at a few million pairs and
// by VALU beyond (seg_emit: 102 us of the 257, 2.4 TB/s of list writes).
// Each view is binned on its own (its slots are one part of the depth sort),
// so that a view's cells fit the tables of the scatter.
// The tiles' lists lie cell by cell; `ranges` says where.
//
// No kernel waits on another work-group.
#include "nxs_internal.h"

#include <algorithm>

namespace nxs {

namespace {

constexpr int kBThreads = 256;
constexpr int kBWaves = kBThreads / 64;
constexpr uint32_t kShortRun = 8;    // slots of more cells are taken by a whole wave
constexpr uint32_t kXcds = 8;
constexpr int kStartThreads = 1024;
constexpr int kMinChunk = 256;
constexpr int64_t kWantChunks = 768;
// Slots from which segments take 256 and 1,024 pairs instead of 64: a wave goes
// through its segment serially (4,096 slots: seg_emit 7.1 us in segments of
// 256, 4.3 of 64), and every segment is a row to sum and scan (200,000 slots:
// the three kernels 18.4 us in segments of 256, 22.8 of 64).
constexpr int64_t kMidFrom = int64_t(1) << 16;
constexpr int64_t kLargeFrom = int64_t(8) << 20;
// a chunk's counts of one cell share a word: pairs in the low bits (a chunk
// has at most 4,096 slots), instances (at most 64 per pair) above
constexpr int kPairBits = 13;
constexpr uint32_t kPairMask = (1u << kPairBits) - 1u;
static_assert(kMaxCellChunk <= 4096 && kMaxCellTiles <= 64, "a chunk's counts fit one word");

template <int NW = kBWaves>   // waves in the work-group
__device__ __forceinline__ uint32_t bin_block_scan(uint32_t x, uint32_t* s_tmp, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan_u32(x);
  if (lane == 63) s_tmp[wid] = incl;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const uint32_t v = s_tmp[w];
    if (w < wid) off += v;
    tot += v;
  }
  __syncthreads();
  *total = tot;
  return off + incl - x;
}

// The chunk of work-group b: XCD b % 8 (work-groups are dealt to the XCDs
// round-robin) takes a contiguous band of chunks, so that the runs which
// neighbouring chunks write for one cell meet in one L2.
__device__ __forceinline__ uint32_t banded_chunk(uint32_t b, uint32_t per) {
  return (b % kXcds) * per + b / kXcds;
}

// A cell's extent: log2 of its 8x8 blocks per row and column, and of a tile's.
struct CellShape {
  int bx, by, ax, ay;
};

// The cells a slot's rectangle covers, in its view's grid of cells.
struct CellSpan {
  uint32_t cx0, cy0, nx, n;   // first cell, cells per row, cells (0: culled)
};
__device__ __forceinline__ CellSpan cell_span(uint2 r, const CellShape& s) {
  CellSpan c{0u, 0u, 1u, 0u};
  if (r.x == 0xFFFFFFFFu) return c;
  c.cx0 = (r.x & 0xFFFFu) >> s.bx;
  c.cy0 = (r.y & 0xFFFFu) >> s.by;
  c.nx = ((r.x >> 16) >> s.bx) - c.cx0 + 1u;
  c.n = c.nx * (((r.y >> 16) >> s.by) - c.cy0 + 1u);
  return c;
}

// The part of the rectangle that lies in cell (cx, cy), in the cell's own
// blocks.  (A cell has at most 64 tiles of at most 4 blocks: its four
// coordinates take at most 16 bits.)
struct LocalRect {
  uint32_t x0, x1, y0, y1;
};
__device__ __forceinline__ LocalRect local_rect(uint2 r, uint32_t cx, uint32_t cy,
                                                const CellShape& c) {
  const uint32_t ox = cx << c.bx, oy = cy << c.by;
  const uint32_t mx = (1u << c.bx) - 1u, my = (1u << c.by) - 1u;
  return {max(r.x & 0xFFFFu, ox) - ox, min((r.x >> 16) - ox, mx),
          max(r.y & 0xFFFFu, oy) - oy, min((r.y >> 16) - oy, my)};
}
__device__ __forceinline__ uint32_t pack_rect(const LocalRect& l, const CellShape& c) {
  return l.x0 | (l.x1 << c.bx) | (l.y0 << (2 * c.bx)) | (l.y1 << (2 * c.bx + c.by));
}

// l / w for l < 2^24 (float, then exact by the +-1 fix-up)
__device__ __forceinline__ uint32_t small_div(uint32_t l, uint32_t w) {
  uint32_t q = (uint32_t)((float)l * __frcp_rn((float)w));
  if (q * w > l) --q;
  if ((q + 1) * w <= l) ++q;
  return q;
}

// What a work-group knows of its chunk: the `col`-th chunk of a view, slots
// [first, end) in the order given, and the view's cells.
struct ChunkOf {
  int64_t first, end;
  uint32_t col, cell0, cells_x, n_cells;
};
__device__ __forceinline__ ChunkOf chunk_of(uint32_t c, uint32_t cpv, uint32_t chunk, int32_t n,
                                            const uint32_t* __restrict__ vis,
                                            const ViewDev* __restrict__ views,
                                            const CellShape& s) {
  ChunkOf k;
  const uint32_t vi = c / cpv;
  k.col = c - vi * cpv;
  k.first = (int64_t)vi * n + (int64_t)k.col * chunk;
  k.end = min(k.first + chunk, (int64_t)vi * n + (vis ? (int64_t)vis[vi] : (int64_t)n));
  const ViewDev& v = views[vi];
  k.cell0 = (uint32_t)v.cell_off;
  k.cells_x = (uint32_t)v.cells_x;
  const int sy = s.by - s.ay;   // tiles
  k.n_cells = k.cells_x * (((uint32_t)v.tiles_y + (1u << sy) - 1u) >> sy);
  return k;
}

template <bool SMALL>
__global__ __launch_bounds__(kBThreads) void cell_count_kernel(
    const uint2* __restrict__ rects, int32_t n, const uint32_t* __restrict__ vis,
    uint32_t nchunks, uint32_t cpv, uint32_t chunk, uint32_t per,
    const ViewDev* __restrict__ views, CellShape shape, uint32_t* __restrict__ counts,
    const Counters* __restrict__ cnt) {
  __shared__ uint32_t h[kViewCells];
  if (cnt->fail) return;
  const uint32_t c = banded_chunk(blockIdx.x, per);
  if (c >= nchunks) return;
  const ChunkOf ck = chunk_of(c, cpv, chunk, n, vis, views, shape);
  const int lane = threadIdx.x & 63;
  for (uint32_t d = threadIdx.x; d < ck.n_cells; d += kBThreads) h[d] = 0u;
  __syncthreads();
  constexpr int kPerT = 2;   // (its loads issued together)
  for (int64_t base = ck.first; base < ck.end; base += kPerT * kBThreads) {
    uint2 r[kPerT];
#pragma unroll
    for (int q = 0; q < kPerT; ++q) {
      const int64_t i = base + q * kBThreads + threadIdx.x;
      r[q] = i < ck.end ? load_rect<SMALL>(rects, i) : make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);
    }
#pragma unroll
    for (int q = 0; q < kPerT; ++q) {
      const CellSpan s = cell_span(r[q], shape);
      auto add = [&](uint2 rc, uint32_t cx, uint32_t cy) {
        const LocalRect l = local_rect(rc, cx, cy, shape);
        const uint32_t w = (l.x1 >> shape.ax) - (l.x0 >> shape.ax) + 1u;   // tiles
        const uint32_t hh = (l.y1 >> shape.ay) - (l.y0 >> shape.ay) + 1u;
        atomicAdd(&h[cy * ck.cells_x + cx], ((w * hh) << kPairBits) | 1u);
      };
      if (s.n <= kShortRun) {
        uint32_t cx = s.cx0, cy = s.cy0;
        for (uint32_t k = 0; k < s.n; ++k) {
          add(r[q], cx, cy);
          if (++cx == s.cx0 + s.nx) {
            cx = s.cx0;
            ++cy;
          }
        }
      }
      uint64_t runs = __ballot(s.n > kShortRun);
      while (runs) {   // (one slot after another, its cells over the lanes)
        const int b = __builtin_ctzll(runs);
        runs &= runs - 1;
        auto from = [&](uint32_t v) {
          return (uint32_t)__builtin_amdgcn_readlane((int)v, b);
        };
        const uint2 rc = make_uint2(from(r[q].x), from(r[q].y));
        const CellSpan t = cell_span(rc, shape);
        for (uint32_t k = lane; k < t.n; k += 64) {
          const uint32_t row = small_div(k, t.nx);
          add(rc, t.cx0 + (k - row * t.nx), t.cy0 + row);
        }
      }
    }
  }
  __syncthreads();
  for (uint32_t d = threadIdx.x; d < ck.n_cells; d += kBThreads)
    counts[(size_t)(ck.cell0 + d) * cpv + ck.col] = h[d];
}

// One work-group per cell: exclusive scan of its pair counts over the chunks,
// in place; totals[d] its pairs, weights[d] its instances.
__global__ __launch_bounds__(kBThreads) void cell_scan_kernel(uint32_t* __restrict__ counts,
                                                              uint32_t nchunks,
                                                              uint32_t* __restrict__ totals,
                                                              uint32_t* __restrict__ weights,
                                                              const Counters* __restrict__ cnt) {
  __shared__ uint32_t s_tmp[kBWaves];
  if (cnt->fail) return;
  uint32_t* row = counts + (size_t)blockIdx.x * nchunks;
  uint32_t running = 0, inst = 0;
  for (uint32_t b = 0; b < nchunks; b += kBThreads * 4) {
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t i = b + threadIdx.x * 4 + q;
      const uint32_t w = i < nchunks ? row[i] : 0u;
      v[q] = w & kPairMask;
      sum += v[q];
      inst += w >> kPairBits;
    }
    uint32_t tot;
    uint32_t ex = bin_block_scan(sum, s_tmp, &tot) + running;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t i = b + threadIdx.x * 4 + q;
      if (i < nchunks) row[i] = ex;
      ex += v[q];
    }
    running += tot;
  }
  uint32_t all;
  (void)bin_block_scan(inst, s_tmp, &all);
  if (threadIdx.x == 0) {
    totals[blockIdx.x] = running;
    weights[blockIdx.x] = all;
  }
}

// Where each cell's pairs, segments (of 2^seg_shift pairs, the last one
// shorter) and instances begin: start[d], d <= n_cells for the first two.  (Every
// cell in one round of loads and scans: 3,094 cells 6.1 us, in rounds of 1,024
// cells 9.)
__global__ __launch_bounds__(kStartThreads) void cell_starts_kernel(
    const uint32_t* __restrict__ totals, const uint32_t* __restrict__ weights, uint32_t n_cells,
    uint32_t seg_shift, uint32_t* __restrict__ pair0, uint32_t* __restrict__ seg0,
    uint32_t* __restrict__ inst0, const Counters* __restrict__ cnt) {
  constexpr int NW = kStartThreads / 64;
  constexpr int PER = kMaxCells / kStartThreads;   // consecutive cells per thread: one round
  static_assert(kMaxCells % kStartThreads == 0, "whole cells per thread");
  __shared__ uint32_t s_tmp[NW];
  if (cnt->fail) return;
  uint32_t v[PER], w[PER], p = 0, g = 0, m = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t d = threadIdx.x * PER + q;
    v[q] = d < n_cells ? totals[d] : 0u;
    w[q] = d < n_cells ? weights[d] : 0u;
    p += v[q];
    g += (v[q] + (1u << seg_shift) - 1u) >> seg_shift;
    m += w[q];
  }
  uint32_t tp, tg, tm;
  p = bin_block_scan<NW>(p, s_tmp, &tp);
  g = bin_block_scan<NW>(g, s_tmp, &tg);
  m = bin_block_scan<NW>(m, s_tmp, &tm);
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const uint32_t d = threadIdx.x * PER + q;
    if (d < n_cells) {
      pair0[d] = p;
      seg0[d] = g;
      inst0[d] = m;
    }
    p += v[q];
    g += (v[q] + (1u << seg_shift) - 1u) >> seg_shift;
    m += w[q];
  }
  if (threadIdx.x == 0) {
    pair0[n_cells] = tp;
    seg0[n_cells] = tg;
  }
}

// kSubPerT consecutive slots per thread at a time, their pairs ranked in windows
// of kWinItems per thread.
template <int kSubPerT, int kWinItems, bool SMALL>
__global__ __launch_bounds__(kBThreads) void cell_scatter_kernel(
    const uint32_t* __restrict__ sorted_slots, const uint2* __restrict__ rects, int32_t n,
    const uint32_t* __restrict__ vis, uint32_t nchunks, uint32_t cpv, uint32_t chunk, uint32_t per,
    const ViewDev* __restrict__ views, CellShape shape, const uint32_t* __restrict__ counts,
    const uint32_t* __restrict__ pair0, uint64_t capacity, uint32_t* __restrict__ pair_slot,
    uint16_t* __restrict__ pair_rect, const Counters* __restrict__ cnt) {
  constexpr int kSub = kBThreads * kSubPerT, kWin = kBThreads * kWinItems;
  constexpr int BINS = kViewCells;
  constexpr int kPer = BINS / kBThreads;   // cells per thread
  __shared__ uint32_t s_off[kSub];
  __shared__ uint32_t s_slot[kSub];
  __shared__ uint2 s_rect[kSub];
  __shared__ __align__(16) uint16_t s_wave[kBWaves][BINS];
  __shared__ uint32_t s_base[BINS];    // next free position of each cell's list
  __shared__ uint32_t s_delta[BINS];   // global minus local start of a window's run
  __shared__ uint32_t s_val[kWin];
  __shared__ uint32_t s_pk[kWin];      // cell << 16 | rectangle within it
  __shared__ uint32_t s_tmp[kBWaves];
  uint16_t* s_owner = reinterpret_cast<uint16_t*>(s_val);   // (dead before s_val is written)

  // (the pairs are at most as many as the instances the buffers hold)
  if (cnt->fail || cnt->total > capacity) return;
  const uint32_t c = banded_chunk(blockIdx.x, per);
  if (c >= nchunks) return;
  const ChunkOf ck = chunk_of(c, cpv, chunk, n, vis, views, shape);
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const int width = 32 - __clz((int)(ck.n_cells - 1u));   // bits of a cell (0: one cell)
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const uint32_t d = t * kPer + k;
    s_base[d] = d < ck.n_cells
                    ? pair0[ck.cell0 + d] + counts[(size_t)(ck.cell0 + d) * cpv + ck.col]
                    : 0u;
  }
  const int64_t end = ck.end;
  for (int64_t base = ck.first; base < end; base += kSub) {
    // kSubPerT consecutive slots per thread
    const int k0 = kSubPerT * t;
    uint32_t a[kSubPerT], e[kSubPerT], total;
    {
      uint2 r[kSubPerT];
      uint32_t slot[kSubPerT], nc[kSubPerT], sum = 0;
#pragma unroll
      for (int q = 0; q < kSubPerT; ++q) {
        const int64_t i = base + k0 + q;
        r[q] = i < end ? load_rect<SMALL>(rects, i) : make_uint2(0xFFFFFFFFu, 0xFFFFFFFFu);
        slot[q] = i < end ? (sorted_slots ? sorted_slots[i] : (uint32_t)i) : 0u;
      }
#pragma unroll
      for (int q = 0; q < kSubPerT; ++q) {
        nc[q] = cell_span(r[q], shape).n;
        sum += nc[q];
      }
      uint32_t ex = bin_block_scan(sum, s_tmp, &total);   // (also: the tables are free)
#pragma unroll
      for (int q = 0; q < kSubPerT; ++q) {
        s_off[k0 + q] = ex;
        s_slot[k0 + q] = slot[q];
        s_rect[k0 + q] = r[q];
        a[q] = ex;
        ex += nc[q];
        e[q] = ex;
      }
    }
    for (uint32_t w0 = 0; w0 < total; w0 += kWin) {
      const uint32_t w1 = min(total, w0 + kWin);
      for (int k = t; k < (int)(sizeof(s_wave) / 16); k += kBThreads)
        reinterpret_cast<uint4*>(&s_wave[0][0])[k] = make_uint4(0u, 0u, 0u, 0u);
      // each slot marks its pairs' places with its index
#pragma unroll
      for (int q = 0; q < kSubPerT; ++q) {
        const bool longrun = e[q] - a[q] > kShortRun;
        if (!longrun)
          for (uint32_t j = max(a[q], w0); j < min(e[q], w1); ++j)
            s_owner[j - w0] = (uint16_t)(k0 + q);
        uint64_t runs = __ballot(longrun);
        while (runs) {
          const int b = __builtin_ctzll(runs);
          runs &= runs - 1;
          const uint32_t ba = (uint32_t)__builtin_amdgcn_readlane((int)a[q], b);
          const uint32_t be = (uint32_t)__builtin_amdgcn_readlane((int)e[q], b);
          const uint16_t bk = (uint16_t)(kSubPerT * (t - lane + b) + q);
          for (uint32_t j = max(ba, w0) + lane; j < min(be, w1); j += 64) s_owner[j - w0] = bk;
        }
      }
      __syncthreads();
      uint32_t dig[kWinItems], val[kWinItems], pk[kWinItems], rank[kWinItems];
      uint32_t lo[kWinItems], hi[kWinItems];
#pragma unroll
      for (int r = 0; r < kWinItems; ++r) {
        const uint32_t li = wid * (64 * kWinItems) + r * 64 + lane;
        const bool valid = w0 + li < w1;
        dig[r] = val[r] = pk[r] = 0u;
        if (valid) {
          const int k = s_owner[li];
          const uint2 rc = s_rect[k];
          const CellSpan s = cell_span(rc, shape);
          const uint32_t l = w0 + li - s_off[k], row = small_div(l, s.nx);
          const uint32_t cx = s.cx0 + (l - row * s.nx), cy = s.cy0 + row;
          dig[r] = cy * ck.cells_x + cx;
          val[r] = s_slot[k];
          pk[r] = (dig[r] << 16) | pack_rect(local_rect(rc, cx, cy, shape), shape);
        }
        const uint64_t m = __ballot(valid);
        lo[r] = (uint32_t)m;
        hi[r] = (uint32_t)(m >> 32);
      }
      match_digits<kWinItems>(dig, width, lo, hi);
#pragma unroll
      for (int r = 0; r < kWinItems; ++r) {
        rank[r] = 0;
        if (w0 + wid * (64 * kWinItems) + r * 64 + lane < w1) {
          const uint32_t before = s_wave[wid][dig[r]];   // the same for every peer
          const uint32_t pos = lanes_below(lo[r], hi[r]);
          rank[r] = before + pos;
          if (pos == 0)
            s_wave[wid][dig[r]] = (uint16_t)(before + (uint32_t)(__popc(lo[r]) + __popc(hi[r])));
        }
      }
      __syncthreads();
      // each cell's run in the window; each wave's count becomes its first
      // place within the run
      {
        uint32_t cn[kPer], sum = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
          cn[k] = 0;
#pragma unroll
          for (int w = 0; w < kBWaves; ++w) cn[k] += s_wave[w][t * kPer + k];
          sum += cn[k];
        }
        uint32_t all;
        uint32_t ex = bin_block_scan(sum, s_tmp, &all);
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
          const int d = t * kPer + k;
          uint32_t run = ex;
#pragma unroll
          for (int w = 0; w < kBWaves; ++w) {
            const uint32_t x = s_wave[w][d];
            s_wave[w][d] = (uint16_t)run;
            run += x;
          }
          const uint32_t g = s_base[d];
          s_delta[d] = g - ex;
          s_base[d] = g + cn[k];
          ex += cn[k];
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kWinItems; ++r) {
        const uint32_t li = wid * (64 * kWinItems) + r * 64 + lane;
        if (w0 + li < w1) {
          const uint32_t at = s_wave[wid][dig[r]] + rank[r];
          s_val[at] = val[r];
          s_pk[at] = pk[r];
        }
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < kWinItems; ++r) {
        const uint32_t i = r * kBThreads + t;
        if (w0 + i < w1) {
          const uint32_t p = s_pk[i];
          const uint32_t g = s_delta[p >> 16] + i;
          pair_slot[g] = s_val[i];
          pair_rect[g] = (uint16_t)p;
        }
      }
      __syncthreads();   // the tables are rebuilt for the next window
    }
  }
}

// The cells' first segments into LDS, eight loads of a thread in flight at a time (a
// load after the other is most of the kernel's time where segments are few: 3,094
// cells of 60 pairs, seg_count 7.6 -> 5.5 us, seg_emit 10.3 -> 9.2).
__device__ __forceinline__ void load_starts(uint32_t* s_seg, const uint32_t* __restrict__ seg0,
                                            uint32_t n_cells) {
  constexpr int PER = 8;
  if (n_cells < kBThreads) {
    if (threadIdx.x <= n_cells) s_seg[threadIdx.x] = seg0[threadIdx.x];
    return;
  }
  for (uint32_t d0 = 0; d0 <= n_cells; d0 += PER * kBThreads) {
    uint32_t v[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) v[q] = seg0[min(d0 + q * kBThreads + threadIdx.x, n_cells)];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const uint32_t d = d0 + q * kBThreads + threadIdx.x;
      if (d <= n_cells) s_seg[d] = v[q];
    }
  }
}

// the cell of segment sg (the last d with s_seg[d] <= sg; sg is below the total)
__device__ __forceinline__ uint32_t cell_of_segment(const uint32_t* s_seg, uint32_t n_cells,
                                                    uint32_t sg) {
  uint32_t lo = 0, hi = n_cells - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (s_seg[mid] <= sg) lo = mid; else hi = mid - 1;
  }
  return __builtin_amdgcn_readfirstlane(lo);   // (sg is the same on every lane)
}

// The blocks of a pair's tiles: those of tile (x, y) of the cell are the bits of
// col[x] & row[y] (row by row within the tile; 0: not covered).
template <int SX, int SY, int AX, int AY>
struct PairBlocks {
  static constexpr int W = 1 << SX, H = 1 << SY, BX = SX + AX, BY = SY + AY;
  uint32_t col[W], row[H];
  __device__ __forceinline__ uint32_t tile(int t) const { return col[t % W] & row[t / W]; }
};
template <int SX, int SY, int AX, int AY>
__device__ __forceinline__ PairBlocks<SX, SY, AX, AY> pair_blocks(uint32_t lr, bool valid) {
  using P = PairBlocks<SX, SY, AX, AY>;
  constexpr int NX = 1 << AX, NY = 1 << AY;   // a tile's blocks
  constexpr uint32_t kMX = (1u << P::BX) - 1u, kMY = (1u << P::BY) - 1u;
  const uint32_t x0 = lr & kMX, x1 = (lr >> P::BX) & kMX;
  const uint32_t y0 = (lr >> (2 * P::BX)) & kMY, y1 = (lr >> (2 * P::BX + P::BY)) & kMY;
  const uint32_t xs = valid ? (uint32_t)((2ull << x1) - (1ull << x0)) : 0u;
  const uint32_t ys = (2u << y1) - (1u << y0);
  P b;
#pragma unroll
  for (int x = 0; x < P::W; ++x) {
    const uint32_t c = (xs >> (x << AX)) & ((1u << NX) - 1u);
    b.col[x] = NY == 2 ? c | (c << NX) : c;
  }
#pragma unroll
  for (int y = 0; y < P::H; ++y) {
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < NY; ++k)
      m |= (ys >> ((y << AY) + k)) & 1u ? ((1u << NX) - 1u) << (k * NX) : 0u;
    b.row[y] = m;
  }
  return b;
}

template <int SX, int SY, int AX, int AY>
__global__ __launch_bounds__(kBThreads) void seg_count_kernel(
    const uint16_t* __restrict__ pair_rect, const uint32_t* __restrict__ pair0,
    const uint32_t* __restrict__ seg0, uint32_t n_cells, uint32_t seg_shift,
    uint32_t* __restrict__ segs, const Counters* __restrict__ cnt) {
  constexpr int NT = 1 << (SX + SY);
  __shared__ uint32_t s_seg[kMaxCells + 1];
  if (cnt->fail) return;
  load_starts(s_seg, seg0, n_cells);
  __syncthreads();
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n_seg = s_seg[n_cells];
  for (uint32_t sg = blockIdx.x * kBWaves + wid; sg < n_seg; sg += gridDim.x * kBWaves) {
    const uint32_t d = cell_of_segment(s_seg, n_cells, sg);
    const PairRange pr = segment_pairs(pair0[d], pair0[d + 1], sg - s_seg[d], seg_shift);
    const uint16_t* rects = pair_rect + pr.first;
    uint32_t n[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) n[t] = 0;
    for (uint32_t p = 0; p < pr.n; p += 256) {
      uint32_t lr[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t i = p + 64 * q + lane;
        lr[q] = i < pr.n ? rects[i] : 0u;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const auto m = pair_blocks<SX, SY, AX, AY>(lr[q], p + 64 * q + lane < pr.n);
#pragma unroll
        for (int t = 0; t < NT; ++t) n[t] += (uint32_t)__popcll(__ballot(m.tile(t) != 0u));
      }
    }
    uint32_t mine = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) mine = lane == t ? n[t] : mine;
    if (lane < NT) segs[(size_t)sg * NT + lane] = mine;
  }
}

// One work-group per cell.  segs[s][t] (instances of tile t in segment s)
// becomes the list position of the first of them, and the tiles' ranges are
// written (a tile without instances keeps the range it was cleared to).
template <int SX, int SY>
__global__ __launch_bounds__(kBThreads) void cell_tiles_kernel(
    const ViewDev* __restrict__ views, int n_views, const uint32_t* __restrict__ seg0,
    const uint32_t* __restrict__ inst0, uint32_t* __restrict__ segs, uint2* __restrict__ ranges,
    const Counters* __restrict__ cnt) {
  constexpr int NT = 1 << (SX + SY);
  constexpr int R = kBThreads / NT;   // segments summed side by side
  __shared__ uint32_t s_sum[R][NT];
  __shared__ uint32_t s_start[NT];
  if (cnt->fail) return;
  const uint32_t d = blockIdx.x;
  const uint32_t first = seg0[d], n_seg = seg0[d + 1] - first;
  if (n_seg == 0) return;
  const int r = threadIdx.x / NT, t = threadIdx.x % NT;
  const uint32_t per = (n_seg + R - 1) / R;
  const uint32_t f = min(n_seg, r * per), l = min(n_seg, f + per);
  uint32_t* col = segs + (size_t)first * NT + t;
  uint32_t sum = 0;
#pragma unroll 8
  for (uint32_t s = f; s < l; ++s) sum += col[(size_t)s * NT];
  s_sum[r][t] = sum;
  __syncthreads();
  uint32_t before = 0, total = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const uint32_t v = s_sum[k][t];
    if (k < r) before += v;
    total += v;
  }
  if (threadIdx.x < 64) {   // (the first wave: lanes below NT hold row 0)
    const uint32_t mine = threadIdx.x < NT ? total : 0u;
    const uint32_t start = inst0[d] + wave_inclusive_scan_u32(mine) - mine;
    if (threadIdx.x < NT) {
      s_start[t] = start;
      int lo = 0, hi = n_views - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if ((uint32_t)views[mid].cell_off <= d) lo = mid; else hi = mid - 1;
      }
      const ViewDev& v = views[lo];
      const uint32_t lc = d - (uint32_t)v.cell_off, cy = lc / (uint32_t)v.cells_x;
      const uint32_t tx = ((lc - cy * (uint32_t)v.cells_x) << SX) + (t & ((1 << SX) - 1));
      const uint32_t ty = (cy << SY) + (t >> SX);
      if (total > 0)   // (only tiles of the view are covered)
        ranges[(uint32_t)v.tile_off + ty * (uint32_t)v.tiles_x + tx] =
            make_uint2(start, start + total);
    }
  }
  __syncthreads();
  uint32_t run = s_start[t] + before;
#pragma unroll 8
  for (uint32_t s = f; s < l; ++s) {
    const uint32_t v = col[(size_t)s * NT];
    col[(size_t)s * NT] = run;
    run += v;
  }
}

template <int SX, int SY, int AX, int AY>
__global__ __launch_bounds__(kBThreads) void seg_emit_kernel(
    const uint32_t* __restrict__ pair_slot, const uint16_t* __restrict__ pair_rect,
    const uint32_t* __restrict__ pair0, const uint32_t* __restrict__ seg0, uint32_t n_cells,
    uint32_t seg_shift, const uint32_t* __restrict__ segs, uint32_t pack_mask,
    uint32_t* __restrict__ list, const Counters* __restrict__ cnt) {
  constexpr int NT = 1 << (SX + SY);
  __shared__ uint32_t s_seg[kMaxCells + 1];
  if (cnt->fail) return;
  load_starts(s_seg, seg0, n_cells);
  __syncthreads();
  const int lane = threadIdx.x & 63, wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n_seg = s_seg[n_cells];
  for (uint32_t sg = blockIdx.x * kBWaves + wid; sg < n_seg; sg += gridDim.x * kBWaves) {
    const uint32_t d = cell_of_segment(s_seg, n_cells, sg);
    const PairRange pr = segment_pairs(pair0[d], pair0[d + 1], sg - s_seg[d], seg_shift);
    const uint32_t first = __builtin_amdgcn_readfirstlane(pr.first);
    const uint32_t n = __builtin_amdgcn_readfirstlane(pr.n);
    const uint32_t* slots = pair_slot + first;
    const uint16_t* rects = pair_rect + first;
    const uint32_t mine = lane < NT ? segs[(size_t)sg * NT + lane] : 0u;
    uint32_t at[NT];   // next list position of each tile (wave-uniform)
#pragma unroll
    for (int t = 0; t < NT; ++t) at[t] = (uint32_t)__builtin_amdgcn_readlane((int)mine, t);
    uint32_t slot_n = 0, lr_n = 0;
    if ((uint32_t)lane < n) {
      slot_n = slots[lane];
      lr_n = rects[lane];
    }
    for (uint32_t p = 0; p < n; p += 64) {
      const uint32_t slot = slot_n;
      const auto m = pair_blocks<SX, SY, AX, AY>(lr_n, p + lane < n);
      if (p + 64 + lane < n) {   // (the next 64 pairs' reads in flight meanwhile)
        slot_n = slots[p + 64 + lane];
        lr_n = rects[p + 64 + lane];
      }
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const uint32_t blocks = m.tile(t);
        const bool in = blocks != 0u;
        const uint64_t who = __ballot(in);
        if (who) {
          if (in)
            list[__builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)who, at[t]))] =
                slot | ((blocks << 28) & pack_mask);
          at[t] += (uint32_t)__popcll(who);
        }
      }
    }
  }
}

}  // namespace

// The smallest cells of which no view has more than kViewCells and the render
// no more than kMaxCells: smaller cells mean more pairs per slot but fewer
// tiles to test per pair.
BinPlan plan_bins(const int32_t* tiles_x, const int32_t* tiles_y, int n_views, int32_t n,
                  int tile_w, int tile_h) {
  const int shapes[3][2] = {{2, 2}, {3, 2}, {3, 3}};
  BinPlan p{};
  p.n = n;
  p.n_views = n_views;
  p.ax = tile_w == 32 ? 2 : tile_w == 16 ? 1 : 0;
  p.ay = tile_h == 16 ? 1 : 0;
  p.pack = (int64_t)n * n_views <= kPackedSlots;
  for (int k = 0; k < 3 && n_views <= kMaxBinViews && !p.n_cells; ++k) {
    p.sx = shapes[k][0];
    p.sy = shapes[k][1];
    int64_t cells = 0, most = 0;
    for (int v = 0; v < n_views; ++v) {
      const int64_t c = (int64_t)((tiles_x[v] + (1 << p.sx) - 1) >> p.sx) *
                        ((tiles_y[v] + (1 << p.sy) - 1) >> p.sy);
      cells += c;
      most = std::max(most, c);
    }
    if (most <= kViewCells && cells <= kMaxCells) p.n_cells = (uint32_t)cells;
  }
  // The rectangles are gathered into depth order, 8 bytes from a random place per
  // slot, and read twice: one word each where every view's blocks allow it (last
  // depth pass, 48M slots 944 -> 769 us, 4M 56 -> 35, 1M 19.1 -> 14; against it,
  // cell_scatter 442 -> 485 us at 48M), two words for larger views.
  p.small = p.n_cells > 0;
  for (int v = 0; v < n_views; ++v)
    p.small = p.small && (tiles_x[v] << p.ax) <= kSmallRectBlocks &&
              (tiles_y[v] << p.ay) <= kSmallRectBlocks;
  const bool large = (int64_t)n * n_views >= kLargeFrom;
  // small renders take small chunks: the scatter is a chain of short steps per
  // chunk (200,000 slots: 9.8 us in chunks of 256, 19.4 in chunks of 1,024);
  // large ones large chunks, which keep the counts few (48M slots: counting,
  // scanning and scattering 661 us in chunks of 4,096, 681 in chunks of 1,024;
  // 4M slots: 147 against 127)
  p.chunk = large ? kMaxCellChunk : 1024;
  while (p.chunk > kMinChunk && (int64_t)n * n_views < kWantChunks * p.chunk) p.chunk /= 2;
  p.seg_shift = large ? 10 : (int64_t)n * n_views >= kMidFrom ? 8 : 6;
  // (a row of a cell's tiles per segment: at most half a word a pair, so that the
  // rows fit where the tile-sorted instances would lie)
  p.seg_shift = std::max(p.seg_shift, (uint32_t)(p.sx + p.sy + 1));
  p.cpv = (uint32_t)((n + p.chunk - 1) / p.chunk);
  return p;
}

size_t bin_counts_words(const BinPlan& p) { return (size_t)p.cpv * p.n_cells; }

// (totals, weights, and the starts of pairs, segments and instances)
size_t bin_cells_words(const BinPlan& p) { return 5 * (size_t)p.n_cells + 2; }

// (pairs <= instances; every cell that has pairs can have a short segment)
size_t bin_seg_words(const BinPlan& p, uint64_t max_pairs) {
  return (size_t)((max_pairs >> p.seg_shift) + std::min<uint64_t>(p.n_cells, max_pairs))
         << (p.sx + p.sy);
}

namespace {

CellShape shape_of(const BinPlan& p) { return {p.sx + p.ax, p.sy + p.ay, p.ax, p.ay}; }

struct CellArrays {
  uint32_t *totals, *weights, *pair0, *seg0, *inst0;
};
CellArrays cell_arrays(const BinPlan& p, const BinBuffers& b) {
  const size_t k = p.n_cells;
  return {b.cells, b.cells + k, b.cells + 2 * k, b.cells + 3 * k + 1, b.cells + 4 * k + 2};
}

template <int SX, int SY, int AX, int AY>
void fine_t(const BinPlan& p, const BinBuffers& b, uint64_t m_plan, const ViewDev* views,
            const Counters* counters, hipStream_t s) {
  const CellArrays a = cell_arrays(p, b);
  // a wave per segment, looping beyond the grid
  const uint64_t segs = (m_plan >> p.seg_shift) + p.n_cells;
  const unsigned grid = (unsigned)std::min<uint64_t>((segs + kBWaves - 1) / kBWaves, kMaxFineGrid);
  hipLaunchKernelGGL((seg_count_kernel<SX, SY, AX, AY>), dim3(grid), dim3(kBThreads), 0, s,
                     b.pair_rect, a.pair0, a.seg0, p.n_cells, p.seg_shift, b.segs, counters);
  hipLaunchKernelGGL((cell_tiles_kernel<SX, SY>), dim3(p.n_cells), dim3(kBThreads), 0, s, views,
                     p.n_views, a.seg0, a.inst0, b.segs, b.ranges, counters);
  hipLaunchKernelGGL((seg_emit_kernel<SX, SY, AX, AY>), dim3(grid), dim3(kBThreads), 0, s,
                     b.pair_slot, b.pair_rect, a.pair0, a.seg0, p.n_cells, p.seg_shift, b.segs,
                     p.pack ? ~kPackMask : 0u, b.list, counters);
}

template <int AX, int AY>
void fine_a(const BinPlan& p, const BinBuffers& b, uint64_t m_plan, const ViewDev* views,
            const Counters* counters, hipStream_t s) {
  if (p.sx == 2)
    fine_t<2, 2, AX, AY>(p, b, m_plan, views, counters, s);
  else if (p.sy == 2)
    fine_t<3, 2, AX, AY>(p, b, m_plan, views, counters, s);
  else
    fine_t<3, 3, AX, AY>(p, b, m_plan, views, counters, s);
}

}  // namespace

void launch_bin_count(const BinPlan& p, const BinBuffers& b, const uint2* rects,
                      const uint32_t* vis, const ViewDev* views, const Counters* counters,
                      hipStream_t s) {
  if (p.n <= 0) return;
  const CellArrays a = cell_arrays(p, b);
  const uint32_t nchunks = p.cpv * p.n_views, per = (nchunks + kXcds - 1) / kXcds;
  hipLaunchKernelGGL(p.small ? cell_count_kernel<true> : cell_count_kernel<false>,
                     dim3(per * kXcds), dim3(kBThreads), 0, s, rects, p.n, vis, nchunks,
                     p.cpv, (uint32_t)p.chunk, per, views, shape_of(p), b.counts, counters);
  hipLaunchKernelGGL(cell_scan_kernel, dim3(p.n_cells), dim3(kBThreads), 0, s, b.counts, p.cpv,
                     a.totals, a.weights, counters);
  hipLaunchKernelGGL(cell_starts_kernel, dim3(1), dim3(kStartThreads), 0, s, a.totals, a.weights,
                     p.n_cells, p.seg_shift, a.pair0, a.seg0, a.inst0, counters);
}

void launch_bin_scatter(const BinPlan& p, const BinBuffers& b, const uint32_t* sorted_slots,
                        const uint2* rects, const uint32_t* vis, const ViewDev* views,
                        uint64_t capacity, const Counters* counters, hipStream_t s) {
  if (p.n <= 0) return;
  const CellArrays a = cell_arrays(p, b);
  const uint32_t nchunks = p.cpv * p.n_views, per = (nchunks + kXcds - 1) / kXcds;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(per * kXcds), dim3(kBThreads), 0, s, sorted_slots, rects,
                       p.n, vis, nchunks, p.cpv, (uint32_t)p.chunk, per, views, shape_of(p), b.counts,
                       a.pair0, capacity, b.pair_slot, b.pair_rect, counters);
  };
  if (p.chunk >= 512)
    go(p.small ? cell_scatter_kernel<2, 4, true> : cell_scatter_kernel<2, 4, false>);
  else
    go(p.small ? cell_scatter_kernel<1, 4, true> : cell_scatter_kernel<1, 4, false>);
}

void launch_bin_tiles(const BinPlan& p, const BinBuffers& b, uint64_t m_plan,
                      const ViewDev* views, const Counters* counters, hipStream_t s) {
  if (p.n <= 0) return;
  if (p.ax == 0)
    fine_a<0, 0>(p, b, m_plan, views, counters, s);
  else if (p.ax == 1)
    fine_a<1, 1>(p, b, m_plan, views, counters, s);
  else
    fine_a<2, 0>(p, b, m_plan, views, counters, s);
}

}  // namespace nxs
