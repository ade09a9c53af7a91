// Depth sort of small views in LDS: a view of at most kLocalMax slots is one
// work-group's, in one kernel instead of the radix sort's nine or twelve.
//
// The keys, relative to their least, are dealt by LDS atomics to 2,048 bins of
// equal steps, in no particular order within a bin, and each key then takes its
// place by comparing itself, and on equal keys its slot, with the few others of
// its bin.  A crowded bin (many equal or nearly equal depths) would make that
// quadratic: such a view is sorted through memory by stable passes of up to 8
// bits (wave matches against per-wave counters).
// Bound by the latency of its dozen steps: 13.5 us for 4,096 slots, where the
// radix sort's nine launches took 35 (a 128x128 render of 4,096 Gaussians
// 112 -> 80 us).  (Larger views dealt to 512 buckets by a sampled table first, and
// each bucket sorted so, measured no faster than the radix sort: 66 against
// 68 us for 1M slots, 124 against 132 us for 4M.)
#include "nxs_internal.h"

namespace nxs {

namespace {

constexpr int kNT = 1024;
constexpr int kDBits = 8;
constexpr int kDBins = 1 << kDBits;
constexpr int kSteps = 2048;        // bins of a bucket
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
  uint32_t run[kDBins];
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

// Sorts the m <= CAP keys of one work-group in LDS and leaves in S.out, in order,
// where each one lay; culled keys are left out.  Returns how many there are, or
// ~0 if some bin is crowded (nothing is sorted then).  The keys are read from
// memory (the bucket is in cache after the first time) rather than kept, which
// leaves registers for all the work-groups LDS has room for.
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
  if (__syncthreads_or(crowded)) return ~0u;
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

// Rectangles of either kind (ProjDev): one moved, and an array's part from i on.
__device__ __forceinline__ void copy_rect(uint2* __restrict__ to, size_t j,
                                          const uint2* __restrict__ from, uint32_t i, bool small) {
  if (small)
    reinterpret_cast<uint32_t*>(to)[j] = reinterpret_cast<const uint32_t*>(from)[i];
  else
    to[j] = from[i];
}
__device__ __forceinline__ uint2* rect_at(uint2* p, size_t i, bool small) {
  return small ? reinterpret_cast<uint2*>(reinterpret_cast<uint32_t*>(p) + i) : p + i;
}

// A bucket through memory (none of its keys culled): passes between
// (k0, v0), where it lies, and (k1, v1), an even number of them, each counting
// the whole bucket and then ranking and moving it kNT ITEMS keys at a time.
template <int ITEMS>
__device__ void sort_memory(uint32_t* k0, uint32_t* v0, uint32_t* k1, uint32_t* v1, int m,
                            const uint2* __restrict__ trect, uint32_t* slots_out,
                            uint2* __restrict__ rect_out, bool small, SortLds& S) {
  constexpr int CAP = kNT * ITEMS, NW = kNT / 64;
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  uint32_t mn = kCulled, mx = 0u;
  for (int i = t; i < m; i += kNT) {
    mn = min(mn, k0[i]);
    mx = max(mx, k0[i]);
  }
  block_range(mn, mx, S.a, S.b);
  const uint32_t top = mx - mn;
  const int bits = top ? 32 - __clz((int)top) : 0;
  int passes = (bits + kDBits - 1) / kDBits;
  passes += passes & 1;
  int shift = 0;
  uint32_t *ks = k0, *vs = v0, *kd = k1, *vd = v1;
  for (int p = 0; p < passes; ++p) {
    const int width = (bits - shift + (passes - p) - 1) / (passes - p);
    const uint32_t mask = (1u << width) - 1u;
    __syncthreads();
    if (t < kDBins) S.run[t] = 0u;
    __syncthreads();
    for (int i = t; i < m; i += kNT) atomicAdd(&S.run[((ks[i] - mn) >> shift) & mask], 1u);
    __syncthreads();
    {
      const uint32_t c = t < kDBins ? S.run[t] : 0u;
      uint32_t all;
      const uint32_t ex = block_scan(c, S.a, &all);
      if (t < kDBins) S.run[t] = ex;
    }
    for (int c0 = 0; c0 < m; c0 += CAP) {
      const int cm = min(CAP, m - c0);
      uint32_t k[ITEMS], v[ITEMS], dig[ITEMS], rank[ITEMS];
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const int li = wid * (64 * ITEMS) + r * 64 + lane;
        k[r] = li < cm ? ks[c0 + li] - mn : 0u;
        v[r] = li < cm ? vs[c0 + li] : 0u;
      }
      clear_waves(S);
      __syncthreads();
      wave_ranks<ITEMS>(k, cm, shift, width, S, dig, rank);
      __syncthreads();
      // (the first position of each wave's digits goes beyond 16 bits: the
      // digit's running start is kept apart from the wave's place in it)
      uint32_t start[ITEMS];
      {
        uint32_t c[NW], sum = 0;
        if (t < kDBins) {
#pragma unroll
          for (int w = 0; w < NW; ++w) {
            c[w] = sum;
            sum += S.wave[w][t];
          }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) start[r] = S.run[dig[r]];
        if (t < kDBins) {
#pragma unroll
          for (int w = 0; w < NW; ++w) S.wave[w][t] = (uint16_t)c[w];
        }
        __syncthreads();
        if (t < kDBins) S.run[t] += sum;
      }
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const int li = wid * (64 * ITEMS) + r * 64 + lane;
        if (li < cm) {
          const uint32_t dst = start[r] + S.wave[wid][dig[r]] + rank[r];
          kd[dst] = k[r] + mn;
          vd[dst] = v[r];
        }
      }
      __syncthreads();
    }
    uint32_t* x = ks;
    ks = kd;
    kd = x;
    x = vs;
    vs = vd;
    vd = x;
    shift += width;
    __threadfence_block();   // this pass's writes before the next pass reads them
  }
  __syncthreads();
  for (int i = t; i < m; i += kNT) {   // (back in v0)
    const uint32_t slot = v0[i];
    slots_out[i] = slot;
    copy_rect(rect_out, i, trect, slot, small);
  }
}

// A view's visible keys and their slots, in slot order, into (key_tmp, slot_tmp);
// returns how many.
__device__ uint32_t compact(const uint32_t* __restrict__ keys, uint32_t first, int m,
                            uint32_t* key_tmp, uint32_t* slot_tmp, uint32_t* s_tmp) {
  uint32_t done = 0;
  for (int i0 = 0; i0 < m; i0 += kNT) {
    const int i = i0 + threadIdx.x;
    const uint32_t k = i < m ? keys[i] : kCulled;
    uint32_t all;
    const uint32_t at = done + block_scan(k != kCulled ? 1u : 0u, s_tmp, &all);
    if (k != kCulled) {
      key_tmp[at] = k;
      slot_tmp[at] = first + (uint32_t)i;
    }
    done += all;
  }
  __threadfence_block();
  __syncthreads();
  return done;
}

// One work-group per view.
__global__ __launch_bounds__(kNT) void depth_local_kernel(
    const uint32_t* __restrict__ depth_key, int32_t n, uint32_t* key_tmp, uint32_t* slot_tmp,
    uint32_t* key_alt, uint32_t* slot_alt, const uint2* __restrict__ trect,
    uint32_t* __restrict__ vis, uint32_t* slots_out, uint2* __restrict__ rect_out, bool small) {
  __shared__ SortLds S;
  const size_t base = (size_t)blockIdx.x * (uint32_t)n;
  const uint32_t* keys = depth_key + base;
  uint32_t seen = sort_lds(keys, n, S);
  if (seen != ~0u) {
#pragma unroll 4
    for (int i = threadIdx.x; i < (int)seen; i += kNT) {
      const uint32_t slot = (uint32_t)base + S.out[i];
      slots_out[base + i] = slot;
      copy_rect(rect_out, base + i, trect, slot, small);
    }
  } else {
    seen = compact(keys, (uint32_t)base, n, key_tmp + base, slot_tmp + base, S.a);
    sort_memory<4>(key_tmp + base, slot_tmp + base, key_alt + base, slot_alt + base, (int)seen,
                   trect, slots_out + base, rect_at(rect_out, base, small), small, S);
  }
  if (threadIdx.x == 0) vis[blockIdx.x] = seen;
}

}  // namespace

void launch_depth_local(const uint32_t* depth_key, const uint2* trect, int32_t n, int n_views,
                        uint32_t* key_tmp, uint32_t* slot_tmp, uint32_t* key_alt,
                        uint32_t* slot_alt, uint32_t* vis, uint32_t* slots_out, uint2* rect_out,
                        bool small, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(depth_local_kernel, dim3(n_views), dim3(kNT), 0, s, depth_key, n, key_tmp,
                     slot_tmp, key_alt, slot_alt, trect, vis, slots_out, rect_out, small);
}

}  // namespace nxs
