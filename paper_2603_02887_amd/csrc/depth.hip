// Depth sort of small views in LDS: a view of at most kLocalMax slots is one
// work-group's, in one kernel instead of the radix sort's nine or twelve launches.
//
// The keys, relative to their least, are dealt by LDS atomics to 2,048 bins of
// equal steps, in no particular order within a bin, and each key then takes its
// place by comparing itself, and on equal keys its slot, with the few others of
// its bin.  A crowded bin (many equal or nearly equal depths) would make that
// quadratic: such a view is sorted by stable passes of up to 8 bits, in LDS too
// (8,192 slots on two planes, a 128x128 render: 89 us, with passes through memory
// 125, with the radix sort 87 to 92; 4,096: 82, 94, 87 to 92).
// Bound by the latency of its dozen steps: 12.2 us for 4,096 slots, where the
// radix sort's twelve launches took 45 (a 128x128 render of 4,096 Gaussians
// 111 -> 84 us).  (Larger views dealt to 512 parts by a sampled table first, and
// each part sorted so, measured no faster than the radix sort: 66 against
// 68 us for 1M slots, 124 against 132 us for 4M.)
#include "nxs_internal.h"

namespace nxs {

namespace {

constexpr int kNT = 1024;
constexpr int kDBits = 8;
constexpr int kDBins = 1 << kDBits;
constexpr int kSteps = 2048;        // bins of a view's keys
constexpr uint32_t kMostInBin = 40; // keys of a bin that are compared with each other
constexpr uint32_t kCulled = 0xFFFFFFFFu;

struct SortLds {
  static constexpr int kWaves = kNT / 64, CAP = kLocalMax;
  uint32_t key[CAP];
  uint16_t idx[CAP];   // where the key lay in the view
  uint16_t out[CAP];   // the sorted view
  union {
    uint32_t bin[kSteps];
    __align__(16) uint16_t wave[kWaves][kDBins];
  };
  uint32_t a[kWaves], b[kWaves];
};

__device__ __forceinline__ uint32_t block_scan(uint32_t x, uint32_t* s_tmp, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t incl = wave_inclusive_scan_u32(x);
  __syncthreads();
  if (lane == 63) s_tmp[wid] = incl;
  __syncthreads();
  uint32_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kNT / 64; ++w) {
    const uint32_t v = s_tmp[w];
    if (w < wid) off += v;
    tot += v;
  }
  *total = tot;
  return off + incl - x;
}

// The least and the greatest of the work-group's values.
__device__ __forceinline__ void block_range(uint32_t& mn, uint32_t& mx, uint32_t* s_a,
                                            uint32_t* s_b) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  mn = wave_min_u32(mn);
  mx = wave_max_u32(mx);
  if (lane == 0) {
    s_a[wid] = mn;
    s_b[wid] = mx;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kNT / 64; ++w) {
    mn = min(mn, s_a[w]);
    mx = max(mx, s_b[w]);
  }
}

// Stable ranks of the items' digits within their wave (S.wave zeroed before);
// items li >= m take part as nothing.
template <int ITEMS>
__device__ __forceinline__ void wave_ranks(const uint32_t (&k)[ITEMS], int m, int shift, int width,
                                           SortLds& S, uint32_t (&dig)[ITEMS],
                                           uint32_t (&rank)[ITEMS]) {
  constexpr int G = ITEMS < 4 ? ITEMS : 4;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t mask = (1u << width) - 1u;
#pragma unroll
  for (int r0 = 0; r0 < ITEMS; r0 += G) {
    uint32_t d[G], lo[G], hi[G];
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const int li = wid * (64 * ITEMS) + (r0 + q) * 64 + lane;
      d[q] = (k[r0 + q] >> shift) & mask;
      const uint64_t v = __ballot(li < m);
      lo[q] = (uint32_t)v;
      hi[q] = (uint32_t)(v >> 32);
    }
    match_digits<G>(d, width, lo, hi);
#pragma unroll
    for (int q = 0; q < G; ++q) {
      const int li = wid * (64 * ITEMS) + (r0 + q) * 64 + lane;
      dig[r0 + q] = d[q];
      rank[r0 + q] = 0;
      if (li < m) {
        const uint32_t before = S.wave[wid][d[q]];   // the same for every peer
        const uint32_t pos = lanes_below(lo[q], hi[q]);
        rank[r0 + q] = before + pos;
        if (pos == 0)
          S.wave[wid][d[q]] = (uint16_t)(before + (uint32_t)(__popc(lo[q]) + __popc(hi[q])));
      }
    }
  }
}

__device__ __forceinline__ void clear_waves(SortLds& S) {
  for (int i = threadIdx.x; i < (int)(sizeof(S.wave) / 16); i += kNT)
    reinterpret_cast<uint4*>(&S.wave[0][0])[i] = make_uint4(0u, 0u, 0u, 0u);
}

// The m <= CAP keys of one work-group, relative to the least (mn; `top` the greatest),
// by stable passes of up to 8 bits between registers and LDS: wave matches against
// per-wave counters.  Culled keys are taken as top + 1, and so come last.  Leaves
// in S.out, in order, where each key lay.
__device__ void sort_passes(const uint32_t* __restrict__ keys, int m, uint32_t mn, uint32_t top,
                            SortLds& S) {
  constexpr int ITEMS = SortLds::CAP / kNT, NW = SortLds::kWaves;
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const int bits = 32 - __clz((int)(top + 1u));
  const int passes = (bits + kDBits - 1) / kDBits;
  uint32_t k[ITEMS], v[ITEMS], dig[ITEMS], rank[ITEMS];
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int li = wid * (64 * ITEMS) + r * 64 + lane;
    const uint32_t x = li < m ? keys[li] : kCulled;
    k[r] = x == kCulled ? top + 1u : x - mn;
    v[r] = (uint32_t)li;
  }
  int shift = 0;
  for (int p = 0; p < passes; ++p) {
    const int width = (bits - shift + (passes - p) - 1) / (passes - p);
    if (p > 0) {
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const int li = wid * (64 * ITEMS) + r * 64 + lane;
        k[r] = li < m ? S.key[li] : 0u;
        v[r] = li < m ? S.idx[li] : 0u;
      }
    }
    clear_waves(S);
    __syncthreads();
    wave_ranks<ITEMS>(k, m, shift, width, S, dig, rank);
    __syncthreads();
    // each wave's count of a digit becomes its first place
    {
      uint32_t c[NW], sum = 0, all;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        c[w] = sum;
        if (t < kDBins) sum += S.wave[w][t];
      }
      const uint32_t ex = block_scan(sum, S.a, &all);
#pragma unroll
      for (int w = 0; w < NW; ++w)
        if (t < kDBins) S.wave[w][t] = (uint16_t)(ex + c[w]);
    }
    __syncthreads();
    const bool last = p == passes - 1;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int li = wid * (64 * ITEMS) + r * 64 + lane;
      if (li < m) {
        const uint32_t at = S.wave[wid][dig[r]] + rank[r];
        if (last) {
          S.out[at] = (uint16_t)v[r];
        } else {
          S.key[at] = k[r];
          S.idx[at] = (uint16_t)v[r];
        }
      }
    }
    __syncthreads();
    shift += width;
  }
}

// Sorts the m <= CAP keys of one work-group in LDS and leaves in S.out, in order,
// where each one lay; culled keys come after the others or not at all.  Returns
// how many others there are.  The keys are read from memory again (they are in
// cache after the first time) rather than kept in registers.
__device__ uint32_t sort_lds(const uint32_t* __restrict__ keys, int m, SortLds& S) {
  const int t = threadIdx.x;
  for (int i = t; i < kSteps; i += kNT) S.bin[i] = 0u;
  uint32_t mn = kCulled, mx = 0u;
#pragma unroll 4
  for (int i = t; i < m; i += kNT) {
    const uint32_t k = keys[i];
    mn = min(mn, k);
    mx = max(mx, k == kCulled ? 0u : k);
  }
  block_range(mn, mx, S.a, S.b);
  if (mn == kCulled) return 0u;   // (all are culled)
  const uint32_t top = mx - mn;
  const int shift = max((top ? 32 - __clz((int)top) : 0) - 11, 0);
#pragma unroll 4
  for (int i = t; i < m; i += kNT) {
    const uint32_t k = keys[i];
    if (k != kCulled) atomicAdd(&S.bin[(k - mn) >> shift], 1u);
  }
  __syncthreads();
  constexpr int kPer = kSteps / kNT;
  uint32_t c[kPer], sum = 0, seen;
  bool crowded = false;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    c[q] = S.bin[kPer * t + q];
    sum += c[q];
    crowded = crowded || c[q] > kMostInBin;
  }
  uint32_t ex = block_scan(sum, S.a, &seen);
  if (__syncthreads_or(crowded)) {
    sort_passes(keys, m, mn, top, S);
    return seen;
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    S.bin[kPer * t + q] = ex;
    ex += c[q];
  }
  __syncthreads();
#pragma unroll 4
  for (int i = t; i < m; i += kNT) {
    const uint32_t k = keys[i];
    if (k == kCulled) continue;
    const uint32_t at = atomicAdd(&S.bin[(k - mn) >> shift], 1u);
    S.key[at] = k;
    S.idx[at] = (uint16_t)i;
  }
  __syncthreads();
  // (a bin's count has become the first place of the next one)
  for (int i = t; i < (int)seen; i += kNT) {
    const uint32_t k = S.key[i], li = S.idx[i], d = (k - mn) >> shift;
    const uint32_t b = d ? S.bin[d - 1] : 0u, e = S.bin[d];
    uint32_t at = b;
    for (uint32_t j = b; j < e; ++j) {
      const uint32_t o = S.key[j];
      if (o < k || (o == k && S.idx[j] < li)) ++at;
    }
    S.out[at] = (uint16_t)li;
  }
  __syncthreads();
  return seen;
}

// A rectangle of either kind (ProjDev), moved.
__device__ __forceinline__ void copy_rect(uint2* __restrict__ to, size_t j,
                                          const uint2* __restrict__ from, uint32_t i, bool small) {
  if (small)
    reinterpret_cast<uint32_t*>(to)[j] = reinterpret_cast<const uint32_t*>(from)[i];
  else
    to[j] = from[i];
}

// One work-group per view.
__global__ __launch_bounds__(kNT) void depth_local_kernel(
    const uint32_t* __restrict__ depth_key, int32_t n, const uint2* __restrict__ trect,
    uint32_t* __restrict__ vis, uint32_t* __restrict__ slots_out, uint2* __restrict__ rect_out,
    bool small) {
  __shared__ SortLds S;
  const size_t base = (size_t)blockIdx.x * (uint32_t)n;
  const uint32_t seen = sort_lds(depth_key + base, n, S);
#pragma unroll 4
  for (int i = threadIdx.x; i < (int)seen; i += kNT) {
    const uint32_t slot = (uint32_t)base + S.out[i];
    slots_out[base + i] = slot;
    copy_rect(rect_out, base + i, trect, slot, small);
  }
  if (threadIdx.x == 0) vis[blockIdx.x] = seen;
}

}  // namespace

void launch_depth_local(const uint32_t* depth_key, const uint2* trect, int32_t n, int n_views,
                        uint32_t* vis, uint32_t* slots_out, uint2* rect_out, bool small,
                        hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(depth_local_kernel, dim3(n_views), dim3(kNT), 0, s, depth_key, n, trect,
                     vis, slots_out, rect_out, small);
}

}  // namespace nxs
