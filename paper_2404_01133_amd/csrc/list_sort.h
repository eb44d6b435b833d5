// Depth order inside tile lists: for lists that are grouped by tile already, in record order.
//
// Sorts of up to 1024 entries run in one wave's registers (bitonic merges, E entries a lane, no LDS and
// no barrier).  Longer lists are cut into chunks of 16384 that a work-group sorts (stable radix passes over
// the depth, in LDS), and list_merge_kernel merges up to 256 sorted runs at a time.
// Keys are (depth, record), unique, so the result does not depend on the network.
#pragma once

#include <type_traits>

#include "radix.h"

namespace gs {
namespace {

constexpr int kListWave = 1024;   // entries a wave sorts
constexpr int kListChunk = kRadixThreads * kRadixMaxItems;  // entries a work-group sorts
constexpr int kListFan = 256;     // runs merged at a time

// value of the lane whose number differs in the bits of M
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  auto dpp = [](uint32_t x, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xF, 0xF, true);
  };
  using std::integral_constant;
  if constexpr (M == 1) return dpp(v, integral_constant<int, 0xB1>{});        // quad [1,0,3,2]
  else if constexpr (M == 2) return dpp(v, integral_constant<int, 0x4E>{});   // quad [2,3,0,1]
  else if constexpr (M == 3) return dpp(v, integral_constant<int, 0x1B>{});   // quad [3,2,1,0]
  else if constexpr (M == 7) return dpp(v, integral_constant<int, 0x141>{});  // half row mirrored
  else if constexpr (M == 15) return dpp(v, integral_constant<int, 0x140>{}); // row mirrored
  else if constexpr (M == 8) return dpp(v, integral_constant<int, 0x128>{});  // row rotated by 8
  else if constexpr (M == 4) return lane_xor<3>(lane_xor<7>(v));
  else return (uint32_t)__shfl_xor((int)v, M, 64);
}
template <int M>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v) {
  return ((uint64_t)lane_xor<M>((uint32_t)(v >> 32)) << 32) | lane_xor<M>((uint32_t)v);
}

template <int E>
__device__ __forceinline__ void order_pair(uint64_t (&k)[E], int i, int j) {
  const uint64_t a = k[i], b = k[j];
  const bool swap = b < a;
  k[i] = swap ? b : a;
  k[j] = swap ? a : b;
}

// strides FROM, FROM / 2, .. 1 inside the lane
template <int E, int FROM>
__device__ __forceinline__ void lane_merge(uint64_t (&k)[E]) {
  if constexpr (FROM >= 1) {
#pragma unroll
    for (int i = 0; i < E; ++i)
      if (!(i & FROM)) order_pair(k, i, i | FROM);
    lane_merge<E, FROM / 2>(k);
  }
}
// sorts of 2, 4, .. E entries inside the lane
template <int E, int SIZE>
__device__ __forceinline__ void lane_sort(uint64_t (&k)[E]) {
  if constexpr (SIZE <= E) {
#pragma unroll
    for (int i = 0; i < E; ++i)
      if (!(i & (SIZE / 2))) order_pair(k, i, i ^ (SIZE - 1));
    lane_merge<E, SIZE / 4>(k);
    lane_sort<E, 2 * SIZE>(k);
  }
}
// strides of D, D / 2, .. 1 lanes
template <int E, int D>
__device__ __forceinline__ void cross_merge(uint64_t (&k)[E], int lane) {
  if constexpr (D >= 1) {
    const bool low = !(lane & D);
#pragma unroll
    for (int e = 0; e < E; ++e) {
      const uint64_t b = lane_xor<D>(k[e]);
      k[e] = (b < k[e]) == low ? b : k[e];
    }
    cross_merge<E, D / 2>(k, lane);
  }
}
// merges of 2, 4, .. 64 lanes' entries: the first step of a merge meets the mirrored entry, so that
// every run is ascending
template <int E, int L>
__device__ __forceinline__ void cross_sort(uint64_t (&k)[E], int lane) {
  if constexpr (L <= 64) {
    const bool low = !(lane & (L / 2));
#pragma unroll
    for (int e = 0; e < (E + 1) / 2; ++e) {
      const uint64_t b = lane_xor<L - 1>(k[E - 1 - e]), c = lane_xor<L - 1>(k[e]);
      k[e] = (b < k[e]) == low ? b : k[e];
      if (e != E - 1 - e) k[E - 1 - e] = (c < k[E - 1 - e]) == low ? c : k[E - 1 - e];
    }
    cross_merge<E, L / 4>(k, lane);
    lane_merge<E, E / 2>(k);
    cross_sort<E, 2 * L>(k, lane);
  }
}

struct ListArgs {
  const uint32_t* ranges;      // [tiles][2]
  const uint32_t* depth_keys;  // [records]
  uint32_t* list;              // pairs' records, grouped by tile; sorted on return
  uint32_t* alt;               // other buffer of the merges
  uint32_t* list_keys;         // their depths meanwhile; then the list's tile ids, as before
  uint32_t* alt_keys;
  uint2* chunks;               // (tile, chunk) of the long lists
  uint32_t* n_chunks;
  int64_t n_tiles;
  uint32_t last_record;        // (no list entry is beyond it unless a wait gave up; keeps reads in bounds then)
  __device__ __forceinline__ uint64_t key(uint32_t rec) const {
    return ((uint64_t)depth_keys[min(rec, last_record)] << 32) | rec;
  }
};

// The wave loads list[0, n), n <= 64 E, and sorts it: k[e] of a lane is entry lane * E + e.
template <int E>
__device__ __forceinline__ void wave_sort(const ListArgs& a, const uint32_t* list, int n, int lane, uint64_t (&k)[E]) {
  uint32_t rec[E];
#pragma unroll
  for (int e = 0; e < E; ++e) rec[e] = e * 64 + lane < n ? list[e * 64 + lane] : 0xFFFFFFFFu;
#pragma unroll
  for (int e = 0; e < E; ++e) k[e] = e * 64 + lane < n ? a.key(rec[e]) : ~0ull;
  lane_sort<E, 2>(k);
  cross_sort<E, 2>(k, lane);
}
template <int E>
__device__ __forceinline__ void wave_sort_list(const ListArgs& a, uint32_t* list, int n, int lane) {
  uint64_t k[E];
  wave_sort<E>(a, list, n, lane, k);
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (lane * E + e < n) list[lane * E + e] = (uint32_t)k[e];
}

// merges of runs of kListChunk * kListFan^p entries that a list of n entries needs
__device__ __forceinline__ int list_passes(uint32_t n) {
  int m = 0;
  for (uint64_t run = kListChunk; run < n; run *= kListFan) ++m;
  return m;
}


// One wave per tile.  Bound by the network's instructions: 64, 128, 256, 512 and 1024 entries take about
// 0.15, 0.35, 0.7, 1.7 and 4 thousand of a wave.  6.3M pairs of eight city views (46K lists, 137 each): 76 us,
// 29M VALU instructions (48 us at full issue); the depth passes this replaces took 192.
__global__ void __launch_bounds__(256) list_sort_kernel(ListArgs a) {
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * 4;
  for (int64_t t = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); t < a.n_tiles;
       t += stride) {
    const uint32_t start = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ranges[2 * t]);
    const int n = __builtin_amdgcn_readfirstlane((int)a.ranges[2 * t + 1]) - (int)start;
    uint32_t* l = a.list + start;
    if (n <= 1) continue;
    if (n <= 64) wave_sort_list<1>(a, l, n, lane);
    else if (n <= 128) wave_sort_list<2>(a, l, n, lane);
    else if (n <= 256) wave_sort_list<4>(a, l, n, lane);
    else if (n <= 512) wave_sort_list<8>(a, l, n, lane);
    else if (n <= kListWave) wave_sort_list<16>(a, l, n, lane);
    else {
      const int c = (n + kListChunk - 1) / kListChunk;
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(a.n_chunks, (uint32_t)c);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
      for (int i = lane; i < c; i += 64) a.chunks[at + i] = make_uint2((uint32_t)t, (uint32_t)i);
    }
  }
}

// A work-group sorts list[0, n), n <= kRadixThreads * ITEMS, into out: four stable passes of 8 bits over
// the depth (the list is in record order), everything in registers and LDS.  (Chunks of 2048 sorted by four
// waves and merged in LDS, merged further by searches: lists of about 4000, 2.3M pairs, 240 us against 75.)
template <int ITEMS>
__device__ __forceinline__ void group_sort_list(RadixLds<8>& lds, const ListArgs& a, const uint32_t* list,
                                                uint32_t* out, uint32_t* out_keys, int n) {
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int slice = wid * 64 * ITEMS + lane;  // item k of the lane is entry slice + 64 k
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) val[k] = slice + k * 64 < n ? list[slice + k * 64] : 0u;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) key[k] = slice + k * 64 < n ? (uint32_t)(a.key(val[k]) >> 32) : 0xFFFFFFFFu;
  uint16_t* hist = lds.wave_hist[wid];
  for (int shift = 0; shift < 32; shift += 8) {
    for (int i = threadIdx.x; i < kRadixWaves * 256 / 2; i += kRadixThreads)
      reinterpret_cast<uint32_t*>(&lds.wave_hist[0][0])[i] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {  // stable rank inside the wave
      const uint32_t d = (key[k] >> shift) & 255u;
      const uint32_t prev = hist[d];
      const uint64_t peers = match_digit<8>(d, ~0ull);
      const uint32_t below = (uint32_t)lanemask_lt_count(peers);
      rank[k] = prev + below;
      if (below == 0) hist[d] = (uint16_t)(prev + (uint32_t)__popcll(peers));
      __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    uint32_t c[kRadixWaves], cnt = 0, total;
    if (threadIdx.x < 256) {
#pragma unroll
      for (int w = 0; w < kRadixWaves; ++w) {
        c[w] = cnt;
        cnt += lds.wave_hist[w][threadIdx.x];
      }
    }
    const uint32_t excl = digit_excl_scan<8>(lds, cnt, &total);
    if (threadIdx.x < 256) {
#pragma unroll
      for (int w = 0; w < kRadixWaves; ++w) lds.wave_hist[w][threadIdx.x] = (uint16_t)(excl + c[w]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const uint32_t at = hist[(key[k] >> shift) & 255u] + rank[k];
      lds.u.s.keys[at] = key[k];
      lds.u.s.vals[at] = val[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      key[k] = lds.u.s.keys[slice + k * 64];
      val[k] = lds.u.s.vals[slice + k * 64];
    }
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k)
    if (slice + k * 64 < n) {
      out[slice + k * 64] = val[k];
      if (out_keys) out_keys[slice + k * 64] = key[k];
    }
  __syncthreads();
}

// Chunks of the long lists, one per work-group, into the buffer from which the list's last merge ends in
// `list` (all of a chunk is read before any of it is written, so that may be the same).
__global__ void __launch_bounds__(kRadixThreads) list_chunk_kernel(ListArgs a) {
  __shared__ RadixLds<8> lds;
  const uint32_t nc = *a.n_chunks;
  for (uint32_t i = blockIdx.x; i < nc; i += gridDim.x) {
    const uint2 c = a.chunks[i];
    const uint32_t start = a.ranges[2 * (int64_t)c.x], len = a.ranges[2 * (int64_t)c.x + 1] - start;
    const uint32_t at = start + c.y * (uint32_t)kListChunk;
    const int n = (int)min((uint32_t)kListChunk, start + len - at);
    const int passes = list_passes(len);
    uint32_t* out = (passes & 1 ? a.alt : a.list) + at;
    uint32_t* keys = passes == 0 ? nullptr : (passes & 1 ? a.alt_keys : a.list_keys) + at;
    if (n <= 2 * kRadixThreads) group_sort_list<2>(lds, a, a.list + at, out, keys, n);
    else if (n <= 4 * kRadixThreads) group_sort_list<4>(lds, a, a.list + at, out, keys, n);
    else if (n <= 8 * kRadixThreads) group_sort_list<8>(lds, a, a.list + at, out, keys, n);
    else group_sort_list<16>(lds, a, a.list + at, out, keys, n);
  }
}

// Merge p: runs of kListChunk * kListFan^p entries, up to kListFan of them into one.  An entry's place is
// its place in its run plus, for every other run of the group, the entries there that come before it
// (binary searches).  Lists that are done by then are left.  Bound by the searches' loads; the depths are
// kept beside the records so that a probe's two loads do not depend on each other (binning of a list of
// 184409: 648 -> 415 us), and an entry has a thread of its own (323 us; four entries a thread 415).  256 runs
// at a time: a launch that finds nothing to do costs 4-5 us of a frame, and one merge covers 4M pairs.
__global__ void __launch_bounds__(1024) list_merge_kernel(ListArgs a, int p) {
  const uint32_t nc = *a.n_chunks;  // (at most 2^30 / 512)
  uint64_t run = kListChunk;
  for (int q = 0; q < p; ++q) run *= kListFan;
  constexpr uint32_t kPart = 1024, kParts = kListChunk / kPart;  // an entry per thread
  for (uint32_t i = blockIdx.x; i < nc * kParts; i += gridDim.x) {
    const uint2 c = a.chunks[i / kParts];
    const uint32_t start = a.ranges[2 * (int64_t)c.x], len = a.ranges[2 * (int64_t)c.x + 1] - start;
    if (run >= len) continue;
    const int left = list_passes(len) - 1 - p;  // merges after this one
    const bool into_list = (left & 1) == 0;
    const uint32_t* src = (into_list ? a.alt : a.list) + start;
    const uint32_t* src_keys = (into_list ? a.alt_keys : a.list_keys) + start;
    uint32_t* dst = (into_list ? a.list : a.alt) + start;
    uint32_t* dst_keys = (into_list ? a.list_keys : a.alt_keys) + start;
    const uint32_t first_at = c.y * (uint32_t)kListChunk + i % kParts * kPart, end = min(len, first_at + kPart);
    for (uint32_t at = first_at + threadIdx.x; at < end; at += kPart) {
      const uint32_t rec = src[at], depth = src_keys[at];
      const uint64_t key = ((uint64_t)depth << 32) | rec;
      const uint64_t own = at / run, first = own / kListFan * kListFan;
      uint64_t pos = first * run + (at - own * run);
      for (uint64_t q = first; q < first + kListFan && q * run < len; ++q) {
        if (q == own) continue;
        uint32_t lo = (uint32_t)(q * run), hi = (uint32_t)((q + 1) * run < len ? (q + 1) * run : len);
        const uint32_t q0 = lo;
        while (lo < hi) {
          const uint32_t mid = lo + (hi - lo) / 2;
          if ((((uint64_t)src_keys[mid] << 32) | src[mid]) < key) lo = mid + 1;
          else hi = mid;
        }
        pos += lo - q0;
      }
      dst[pos] = rec;
      dst_keys[pos] = left == 0 ? c.x : depth;  // (c.x: the tile)
    }
  }
}

}  // namespace
}  // namespace gs
