// Depth order inside tile lists: for lists that are grouped by tile already, in record order.
//
// Sorts of up to 1024 entries run in one wave's registers (bitonic merges, E entries a lane, no LDS and
// no barrier).  Longer lists are cut into chunks of 16384 that a work-group sorts (stable radix passes over
// the depth, in LDS), and list_merge_kernel merges up to 256 sorted runs at a time, linear in the list's length.
// Keys are (depth, record), unique, so the result does not depend on the network.
#pragma once

#include <type_traits>

#include "radix.h"

namespace gs {
namespace {

constexpr int kListWave = 1024;   // entries a wave sorts
constexpr int kListChunk = kRadixThreads * kRadixMaxItems;  // entries a work-group sorts
constexpr int kListFan = 256;     // runs merged at a time
constexpr int kListSearched = 6;  // runs up to which an entry searches the others
constexpr int kListPart = 4 * kRadixThreads;  // merged entries a work-group makes

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
  uint2* chunks;               // (tile, chunk) of the long lists, [max_chunks]: those of lists of several chunks
  uint32_t* n_chunks;          // from the front, those of a single one from the back; how many of each
  uint32_t max_chunks;
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
      if (lane == 0) at = atomicAdd(a.n_chunks + (c == 1), (uint32_t)c);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
      // (there is room for all, but if a wait gave up the ranges of several tiles may overlap)
      for (uint32_t i = lane; i < (uint32_t)c && at + i < a.max_chunks; i += 64)
        a.chunks[c == 1 ? a.max_chunks - 1u - at : at + i] = make_uint2((uint32_t)t, i);
    }
  }
}

// A work-group sorts n <= kRadixThreads * ITEMS entries by depth: four stable passes of 8 bits, everything in
// registers and LDS.  load(key, val, slice) reads item k of the calling lane, entry slice + 64 k, for all k (past
// n: key 0xFFFFFFFF); store(i, key, val) gets entry i.  (Chunks of 2048 sorted by four waves and merged in LDS,
// merged further by searches: lists of about 4000, 2.3M pairs, 240 us against 75.)
template <int ITEMS, class Lds, class Load, class Store>
__device__ __forceinline__ void group_sort(Lds& lds, int n, Load load, Store store) {
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int slice = wid * 64 * ITEMS + lane;
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
  load(key, val, slice);
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
    if (slice + k * 64 < n) store(slice + k * 64, key[k], val[k]);
  __syncthreads();
}

// with as many items per thread as n entries need; load is called with their number
template <class Load, class Store>
__device__ __forceinline__ void group_sort_n(RadixLds<8>& lds, int n, Load load, Store store) {
  if (n <= 2 * kRadixThreads) group_sort<2>(lds, n, load, store);
  else if (n <= 4 * kRadixThreads) group_sort<4>(lds, n, load, store);
  else if (n <= 8 * kRadixThreads) group_sort<8>(lds, n, load, store);
  else group_sort<16>(lds, n, load, store);
}

// Chunks of the long lists, one per work-group, into the buffer from which the list's last merge ends in
// `list` (all of a chunk is read before any of it is written, so that may be the same).  A chunk is in record
// order, so that stable passes over the depth suffice.
__global__ void __launch_bounds__(kRadixThreads) list_chunk_kernel(ListArgs a) {
  __shared__ RadixLds<8> lds;
  const uint32_t several = min(a.n_chunks[0], a.max_chunks), nc = several + min(a.n_chunks[1], a.max_chunks);
  for (uint32_t i = blockIdx.x; i < nc; i += gridDim.x) {
    const uint2 c = a.chunks[i < several ? i : a.max_chunks - 1u - (i - several)];
    const uint32_t start = a.ranges[2 * (int64_t)c.x], len = a.ranges[2 * (int64_t)c.x + 1] - start;
    const uint32_t at = start + c.y * (uint32_t)kListChunk;
    const int n = (int)min((uint32_t)kListChunk, start + len - at);
    const int passes = list_passes(len);
    const uint32_t* list = a.list + at;
    uint32_t* out = (passes & 1 ? a.alt : a.list) + at;
    uint32_t* keys = passes == 0 ? nullptr : (passes & 1 ? a.alt_keys : a.list_keys) + at;
    group_sort_n(
        lds, n,
        [&](auto& key, auto& val, int slice) {
          constexpr int kItems = sizeof(key) / sizeof(key[0]);
#pragma unroll
          for (int k = 0; k < kItems; ++k) val[k] = slice + k * 64 < n ? list[slice + k * 64] : 0u;
#pragma unroll
          for (int k = 0; k < kItems; ++k)
            key[k] = slice + k * 64 < n ? (uint32_t)(a.key(val[k]) >> 32) : 0xFFFFFFFFu;
        },
        [&](int j, uint32_t key, uint32_t val) {
          out[j] = val;
          if (keys) keys[j] = key;
        });
  }
}

// Sorted runs that are merged into one: run q is entries [q * run, q * run + length(q)) from `keys` and `vals`.
struct MergeGroup {
  const uint32_t* keys;
  const uint32_t* vals;
  uint32_t run, total;
  int runs;  // 1 .. kListFan
  __device__ __forceinline__ uint32_t length(int q) const { return min(run, total - (uint32_t)q * run); }
};

// Entries of every run (at[j][q]) among the first n[j] <= total of the merged order, for two n side by side; the
// whole work-group.  The depth of merged entry n is found from its high bits to its low ones: kRadixThreads
// threads, one per run and value of the next bits, count the smaller depths of the run by a search between the
// places found so far.  Entries of that depth itself are taken run after run, which is record order.
struct MergeSplit {  // in LDS
  uint32_t lo[2][kListFan];  // entries of the run below the depths left
  uint32_t hi[2][kListFan];  // and below or among them
  uint32_t sum[2][256];      // per value of the bits, over the runs
  uint32_t place[2][kRadixThreads];
  uint32_t range[2];         // smallest and largest depth
};
using MergeLds = RadixLds<8, kListPart / kRadixThreads>;
__device__ __forceinline__ void merge_split(MergeLds& lds, const MergeGroup& g, const uint32_t (&n)[2],
                                            uint32_t (*at)[kListFan]) {
  static_assert(sizeof(MergeSplit) <= sizeof(lds.u.words), "fits where the entries go later");
  MergeSplit& m = *reinterpret_cast<MergeSplit*>(lds.u.words);
  const int tid = threadIdx.x;
  int lr = 2;  // log2 of the threads per value: the runs, rounded up
  while ((1 << lr) < g.runs) ++lr;
  const int most = 10 - lr < 8 ? 10 - lr : 8;  // bits per round
  const int q = tid & ((1 << lr) - 1), c = tid >> lr;
  if (tid == 0) {
    m.range[0] = 0xFFFFFFFFu;
    m.range[1] = 0u;
  }
  __syncthreads();
  if (tid < g.runs) {
    const uint32_t len = g.length(tid);
    const uint32_t* k = g.keys + (size_t)tid * g.run;
    m.lo[0][tid] = m.lo[1][tid] = 0u;
    m.hi[0][tid] = m.hi[1][tid] = len;
    atomicMin(&m.range[0], k[0]);
    atomicMax(&m.range[1], k[len - 1]);
  }
  __syncthreads();
  const uint32_t differ = m.range[0] ^ m.range[1];
  int shift = differ ? 32 - __clz(differ) : 0;
  uint32_t depth[2];  // the bits known so far
  depth[0] = depth[1] = shift < 32 ? m.range[0] >> shift << shift : 0u;
  while (shift > 0) {
    const int b = min(most, shift);
    shift -= b;
    if (tid < 512) m.sum[tid >> 8][tid & 255] = 0u;
    __syncthreads();
    const bool mine = q < g.runs && c < (1 << b);
    uint32_t x[2] = {0u, 0u};
    if (mine) {
      uint32_t end[2];
      const uint32_t* k = g.keys + (size_t)q * g.run;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        x[j] = m.lo[j][q];
        end[j] = c > 0 ? m.hi[j][q] : x[j];
      }
      while ((x[0] < end[0]) | (x[1] < end[1])) {  // (both searches' loads in flight together)
        uint32_t mid[2], key[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          mid[j] = x[j] + (end[j] - x[j]) / 2;
          key[j] = x[j] < end[j] ? k[mid[j]] : 0u;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const bool less = key[j] < (depth[j] | ((uint32_t)c << shift));
          if (x[j] < end[j]) {
            x[j] = less ? mid[j] + 1 : x[j];
            end[j] = less ? end[j] : mid[j];
          }
        }
      }
      m.place[0][tid] = x[0];
      m.place[1][tid] = x[1];
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (lr >= 6) {  // (one value per wave)
        const int w = wave_incl_scan((int)x[j]);
        if ((tid & 63) == 63 && c < (1 << b)) atomicAdd(&m.sum[j][c], (uint32_t)w);
      } else if (mine) {
        atomicAdd(&m.sum[j][c], x[j]);
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int pick = __syncthreads_count(tid < (1 << b) && m.sum[j][tid & 255] <= n[j]) - 1;  // (sum[0] <= n)
      if (tid < g.runs) {
        m.lo[j][tid] = m.place[j][(pick << lr) | tid];
        if (pick + 1 < (1 << b)) m.hi[j][tid] = m.place[j][((pick + 1) << lr) | tid];
      }
      depth[j] |= (uint32_t)pick << shift;
    }
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t below = tid < g.runs ? m.lo[j][tid] : 0u;
    const uint32_t same = tid < g.runs && m.hi[j][tid] > below ? m.hi[j][tid] - below : 0u;
    uint32_t all_below, all_same;
    digit_excl_scan<8>(lds, below, &all_below);
    const uint32_t before = digit_excl_scan<8>(lds, same, &all_same);
    const uint32_t left = n[j] - all_below;  // entries of the depth itself
    if (tid < g.runs) at[j][tid] = below + (left > before ? min(left - before, same) : 0u);
  }
  __syncthreads();
}

// Merge p: runs of kListChunk * kListFan^p entries, up to kListFan of them into one.  Of few runs, an entry per
// thread: its place is its place in its run plus, for every other run, the entries there that come before it
// (binary searches).  Of more, a work-group per kListPart entries of the result: the splits at its ends say
// which entries of every run it holds, and it sorts them as a chunk is sorted (run after run they are in record
// order among equal depths), so that a merge is linear in the list.  256 runs at a time: a launch that finds
// nothing to do costs 4-5 us of a frame, and one merge covers 4M pairs.
// Bound by the dependent loads of the searches.  Whole binning of one list, us, runs searched by every entry ->
// by splits: 3 runs 105 -> 130, 6 runs 114 -> 137, 12 runs 146 -> 155, 24 runs 238 -> 179, 100 runs 2215 -> 319, 4M
// entries 13935 -> 649; many lists, the longest of 3 runs 186 -> 214, of 12 runs 323 -> 239.  Hence the line at
// six runs.  (Parts of 16384 entries, one per chunk: 105 us for the merge of 12 runs against 87, most of a
// list's chunks then on a few CUs.)
struct MergeArgs {  // of one chunk
  MergeGroup g;
  uint32_t* dst;       // as g's arrays, merged
  uint32_t* dst_keys;
  uint32_t first;      // place of the chunk in the group
  uint32_t tile;
  bool last_merge;
  __device__ __forceinline__ void store(uint32_t at, uint32_t key, uint32_t val) const {
    dst[at] = val;
    dst_keys[at] = last_merge ? tile : key;
  }
};
// false: the list of chunk c is merged already
__device__ __forceinline__ bool merge_args(const ListArgs& a, uint2 c, uint32_t run, int p, MergeArgs& m) {
  const uint32_t start = a.ranges[2 * (int64_t)c.x], len = a.ranges[2 * (int64_t)c.x + 1] - start;
  if (run >= len) return false;
  const uint64_t span = (uint64_t)run * kListFan, at = (uint64_t)c.y * kListChunk;
  const uint32_t base = (uint32_t)(at / span * span);  // of the group in the list
  const uint32_t total = (uint32_t)min(span, (uint64_t)(len - base));
  const int left = list_passes(len) - 1 - p;  // merges after this one
  const bool into_list = (left & 1) == 0;
  m.g = MergeGroup{(into_list ? a.alt_keys : a.list_keys) + start + base, (into_list ? a.alt : a.list) + start + base,
                   run, total, (int)((total + run - 1) / run)};
  m.dst = (into_list ? a.list : a.alt) + start + base;
  m.dst_keys = (into_list ? a.list_keys : a.alt_keys) + start + base;
  m.first = (uint32_t)at - base;
  m.tile = c.x;
  m.last_merge = left == 0;
  return true;
}

// entry `at` of the group to its place
__device__ __forceinline__ void merge_searched(const MergeArgs& m, uint32_t at) {
  const uint32_t key = m.g.keys[at], own = at / m.g.run;
  uint32_t pos = at - own * m.g.run;
  for (uint32_t q = 0; q < (uint32_t)m.g.runs; ++q) {
    if (q == own) continue;
    const uint32_t* k = m.g.keys + (size_t)q * m.g.run;
    const uint32_t bound = key + (q < own ? 1u : 0u);  // (equal depths of an earlier run come before)
    uint32_t lo = 0, hi = m.g.length((int)q);
    while (lo < hi) {
      const uint32_t mid = lo + (hi - lo) / 2;
      if (k[mid] < bound) lo = mid + 1;
      else hi = mid;
    }
    pos += lo;
  }
  m.store(min(pos, m.g.total - 1u), key, m.g.vals[at]);  // (in bounds also if a wait gave up)
}

// entries [first, last) of the result
__device__ __forceinline__ void merge_sorted(MergeLds& lds, uint32_t (*s_at)[kListFan], const MergeArgs& m,
                                             uint32_t first, uint32_t last) {
  static_assert(kListFan == 256, "one digit_excl_scan holds the runs");
  const int runs = m.g.runs;
  const uint32_t ends[2] = {first, last};
  merge_split(lds, m.g, ends, s_at);
  const uint32_t q_first = threadIdx.x < runs ? s_at[0][threadIdx.x] : 0u;
  const uint32_t q_n = threadIdx.x < runs ? s_at[1][threadIdx.x] - q_first : 0u;
  uint32_t sum;
  const uint32_t q_at = digit_excl_scan<8>(lds, q_n, &sum);
  if (threadIdx.x < kListFan) {
    lds.goff[threadIdx.x] = q_at;                                    // first of the entries from run q
    lds.delta[threadIdx.x] = threadIdx.x * m.g.run + q_first - q_at;  // its place in the group less that
  }
  __syncthreads();
  const int n = (int)(last - first);
  group_sort<kListPart / kRadixThreads>(
      lds, n,
      [&](auto& key, auto& val, int slice) {
        constexpr int kItems = sizeof(key) / sizeof(key[0]);
        uint32_t from[kItems];
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
          const uint32_t e = (uint32_t)(slice + k * 64);
          int q = 0;  // last run whose entries begin at or before e
          for (int step = kListFan / 2; step > 0; step >>= 1)
            if (q + step < runs && lds.goff[q + step] <= e) q += step;
          from[k] = min(lds.delta[q] + e, m.g.total - 1u);  // (in bounds also if a wait gave up)
        }
#pragma unroll
        for (int k = 0; k < kItems; ++k) {
          const bool in = slice + k * 64 < n;
          key[k] = in ? m.g.keys[from[k]] : 0xFFFFFFFFu;
          val[k] = in ? m.g.vals[from[k]] : 0u;
        }
      },
      [&](int j, uint32_t key, uint32_t val) { m.store(first + (uint32_t)j, key, val); });
}

__global__ void __launch_bounds__(kRadixThreads, 8) list_merge_kernel(ListArgs a, int p) {
  __shared__ MergeLds lds;
  __shared__ uint32_t s_at[2][kListFan];
  const uint32_t nc = min(a.n_chunks[0], a.max_chunks);  // (at most 2^30 / 8192)
  uint32_t run = kListChunk;
  for (int q = 0; q < p; ++q) run *= kListFan;
  constexpr uint32_t kEntries = kListChunk / kRadixThreads, kParts = kListChunk / kListPart;
  MergeArgs m;
  for (uint32_t i = blockIdx.x; i < nc * kEntries; i += gridDim.x) {
    if (!merge_args(a, a.chunks[i / kEntries], run, p, m) || m.g.runs > kListSearched) continue;
    const uint32_t at = m.first + i % kEntries * kRadixThreads + threadIdx.x;
    if (at < m.g.total) merge_searched(m, at);
  }
  for (uint32_t i = blockIdx.x; i < nc * kParts; i += gridDim.x) {
    if (!merge_args(a, a.chunks[i / kParts], run, p, m) || m.g.runs <= kListSearched) continue;
    const uint32_t first = m.first + i % kParts * kListPart;
    if (first < m.g.total) merge_sorted(lds, s_at, m, first, min(first + (uint32_t)kListPart, m.g.total));
  }
}

}  // namespace
}  // namespace gs
