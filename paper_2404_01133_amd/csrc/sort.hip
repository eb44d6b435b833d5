// Tile binning: (tile, depth, record) ordering of the projected Gaussians, in one of two
// orders of work (lists_by_tile says which, and why).
//
// Depth first.  The (tile | depth) key of every (tile, Gaussian) pair is sorted by a
// stable least-significant-digit radix sort.  Its low (depth) digits do not depend on
// the tile, so those passes run once per visible record, before the pairs are
// duplicated; only the tile digits run over the pairs.
//   1. hist      digit histograms of the visible records' depth keys
//   2. 4 passes  stable radix sort by the 32-bit depth key (ties keep record order);
//                the first one reads every selected record and keeps the visible
//                ones (compaction)
//   3. emit      the sorted records' footprint words gathered, their tile counts
//                scanned (one look-back word per work-group tile) and one
//                (view*tiles + tile, record) pair written per tile of each
//                footprint, with the histograms of the tile digits
//   4. passes    stable radix sort by tile id (ceil(bits / 9) passes)
//   5. ranges    [start, end) of every tile
// By tile.  Stages 1 and 2 fall away, stage 3 emits in record order (the zero fill in
// front of it sums the records' tile counts, so there is no look-back), and
//   6. lists     every list is sorted by (depth, record) for itself
// Either way the result equals a sort by (tile, depth, record id).
//
// The radix passes are single-pass with decoupled
// look-back: work-groups take tile ids from an atomic counter in launch order,
// publish their local aggregate, then walk back over predecessors' published
// values.  A work-group
// only waits on tiles claimed before its own, so the waits always end; each
// wait is still bounded (kSpinLimit) and raises GS_FLAG_WAIT if it gives up.
// Every device size is read from the counts array, so nothing here needs a
// host synchronisation and the whole stage can be captured in a HIP graph.
#include <mutex>

#include "list_sort.h"
#include "radix.h"

namespace gs {
namespace {

constexpr int kMaxTilePasses = 4;       // digits of a tile id (below 2^31) at up to 9 bits
constexpr int kTileDigits = 512;        // words of one tile-digit histogram
constexpr int kHistItems = 8;           // records per thread of the depth histogram
constexpr uint32_t kBigFootprint = 16;    // records touching more tiles are emitted by a wave each,
constexpr uint32_t kHugeFootprint = 512;  // with more than this by a work-group
// emit_kernel's work-groups all finish at about the same time and each adds its
// tile-digit histogram to device memory, so a single copy would take ~2000
// same-address atomics per word in a row.  They add into kTileHistCopies
// partial copies instead (copy blockIdx.x mod kTileHistCopies; copy 0 is the
// histogram the radix passes read), and emit_big_kernel, which runs next, folds
// copies 1.. into copy 0.
constexpr int kTileHistCopies = 8;
constexpr int64_t kTileHistWords = kMaxTilePasses * kTileDigits;  // one copy

// Records per thread of the emission: a small input still spreads over the chip (records with many
// tiles make a work-group's share long), a large one keeps the look-back short.
constexpr int kEmitMaxItems = 8;
__host__ __device__ constexpr int emit_items(int64_t n) {
  return n <= (int64_t)1 << 16 ? 1 : n <= (int64_t)1 << 19 ? 4 : kEmitMaxItems;
}
__host__ __device__ constexpr int64_t emit_tiles(int64_t n) {
  const int64_t t = (int64_t)kThreads * emit_items(n);
  return (n + t - 1) / t;
}
// upper bound of emit_tiles(m) over all m <= n
__host__ __device__ constexpr int64_t emit_tiles_bound(int64_t n) {
  int64_t t = emit_tiles(n);
  const int64_t b = emit_tiles(n < ((int64_t)1 << 19) ? n : (int64_t)1 << 19);
  const int64_t c = emit_tiles(n < ((int64_t)1 << 16) ? n : (int64_t)1 << 16);
  t = b > t ? b : t;
  return c > t ? c : t;
}

// ---------------------------------------------------------------------------
// zero fill of the small fixed state (counters, histograms), of the look-back
// words of the depth passes and the emission (sized by the selected records) and
// of the tile passes (sized by the pair capacity: the pair count is not known
// yet), and of the tile ranges
// ---------------------------------------------------------------------------
struct ClearArgs {
  uint32_t* fixed;
  int64_t fixed_words;
  uint32_t* dstatus;  // [tile][4][256]
  uint64_t* estatus;  // [tile]
  uint32_t* pstatus;
  int64_t pstatus_words;
  uint32_t* ranges;
  int64_t range_words;
  // by tile: pairs of every emission tile (into estatus) and, per group of tiles, pairs and visible records
  const int32_t* tiles_touched;
  uint64_t* group_pairs;
  uint32_t* group_visible;
};

// Groups of emission tiles, at most kEmitGroups of equal size.
constexpr int64_t kEmitGroups = 2048;
__device__ __forceinline__ int64_t emit_group_tiles(int64_t ntiles) { return (ntiles + kEmitGroups - 1) / kEmitGroups; }

// sum of x over the work-group, to every thread; s: a word per wave
__device__ __forceinline__ uint64_t group_sum(uint64_t x, uint64_t* s) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) x += (uint64_t)__shfl_xor((unsigned long long)x, d, 64);
  if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = x;
  __syncthreads();
  uint64_t sum = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) sum += s[w];
  __syncthreads();
  return sum;
}

// What the emission in record order needs to know of the records in front of a tile: read once here, beside
// the zero fill, so that no emission tile waits for another.
__device__ __forceinline__ void emit_sums(const ClearArgs& a, int64_t n, uint64_t* s) {
  const int items = emit_items(n);
  const int64_t ntiles = emit_tiles(n), per = emit_group_tiles(ntiles);
  for (int64_t g = blockIdx.x; g * per < ntiles; g += gridDim.x) {
    uint64_t pairs = 0, visible = 0;
    for (int64_t t = g * per; t < (g + 1) * per && t < ntiles; ++t) {
      uint64_t sum = 0;
      for (int k = 0; k < items; ++k) {
        const int64_t i = (t * items + k) * kThreads + threadIdx.x;
        const int32_t c = i < n ? a.tiles_touched[i] : 0;
        sum += c > 0 ? (uint64_t)c : 0ull;
        visible += c > 0 ? 1ull : 0ull;
      }
      sum = group_sum(sum, s);
      if (threadIdx.x == 0) a.estatus[t] = sum;
      pairs += sum;
    }
    visible = group_sum(visible, s);
    if (threadIdx.x == 0) {
      a.group_pairs[g] = pairs;
      a.group_visible[g] = (uint32_t)visible;
    }
  }
}

template <bool BY_TILE>
__global__ void __launch_bounds__(kThreads) clear_front_kernel(ClearArgs a, int64_t* counts, int64_t cap) {
  const int64_t n = count_clamped(counts, GS_COUNT_RECORDS, cap);
  const int64_t dwords = BY_TILE ? 0 : radix_tiles(n) * 4 * kRadix, ewords = BY_TILE ? 0 : emit_tiles(n);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i0 == 0) {
    counts[GS_COUNT_VISIBLE] = 0;  // (no record: no tile writes them)
    counts[GS_COUNT_PAIRS] = 0;
  }
  for (int64_t i = i0; i < a.fixed_words; i += stride) a.fixed[i] = 0u;
  for (int64_t i = i0; i < dwords; i += stride) a.dstatus[i] = 0u;
  for (int64_t i = i0; i < ewords; i += stride) a.estatus[i] = 0ull;
  for (int64_t i = i0; i < a.pstatus_words; i += stride) a.pstatus[i] = 0u;
  for (int64_t i = i0; i < a.range_words; i += stride) a.ranges[i] = 0u;
  if constexpr (BY_TILE) {
    __shared__ uint64_t s_sum[kThreads / 64];
    emit_sums(a, n, s_sum);
  }
}

// ---------------------------------------------------------------------------
// 1. histograms of the visible records' depth digits (all four passes); the
//    work-groups finish together, so their device atomics are spread over
//    kDepthHistCopies partial copies (copy 0 is the histogram itself; each pass
//    adds the others to its digit)
// ---------------------------------------------------------------------------
constexpr int kDepthHistCopies = 8;
static_assert(kDepthHistCopies - 1 <= kRadixMaxCopies, "a pass sums them");
constexpr int64_t kDepthHistWords = 4 * kRadix;

// Histogram adds of a wave whose lanes often share a digit.  Depth keys are
// float bits and a wave holds neighbouring Gaussians, so the top digit (sign and
// exponent) and the next one take a few values per wave; plain LDS atomics on
// them serialise on one address.  match_add: each lane finds the lanes with its
// digit with eight ballots (a fixed cost whatever the distribution) and the
// lowest of them adds their count.  top_add: one round per distinct top digit
// in the wave (sign and exponent of depths within a wave: one or two values).
__device__ __forceinline__ void match_add(bool valid, uint32_t d, uint32_t* h) {
  uint64_t peers = __ballot(valid);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const bool b = (d >> bit) & 1u;
    const uint64_t m = __ballot(b);
    peers &= b ? m : ~m;
  }
  if (valid && lanemask_lt_count(peers) == 0) atomicAdd(&h[d], (uint32_t)__popcll(peers));
}

__device__ __forceinline__ void top_add(bool valid, uint32_t d, uint32_t* h) {
  const int lane = threadIdx.x & 63;
  uint64_t left = __ballot(valid);
  while (left) {
    const int leader = (int)__builtin_ctzll(left);
    const uint32_t dl = (uint32_t)__builtin_amdgcn_readlane((int)d, leader);
    const uint64_t m = __ballot(valid && d == dl);
    if (lane == leader) atomicAdd(&h[dl], (uint32_t)__popcll(m));
    left &= ~m;
  }
}

__global__ void __launch_bounds__(kThreads) depth_hist_kernel(const int32_t* __restrict__ tiles_touched,
                                                              const uint32_t* __restrict__ depth_keys, int64_t cap,
                                                              const int64_t* counts, uint32_t* __restrict__ hist,
                                                              uint32_t* __restrict__ hist_extra) {
  __shared__ uint32_t s_hist[4][kRadix];
  const int64_t n = count_clamped(counts, GS_COUNT_RECORDS, cap);
  const int64_t per_block = (int64_t)kThreads * kHistItems;
  const int64_t nblocks = (n + per_block - 1) / per_block;
  if ((int64_t)blockIdx.x >= nblocks) return;
  for (int i = threadIdx.x; i < 4 * kRadix; i += kThreads) (&s_hist[0][0])[i] = 0u;
  __syncthreads();
  for (int64_t b = blockIdx.x; b < nblocks; b += gridDim.x) {
    // every load of the block's share in flight together (a culled record's key is read and dropped)
    int32_t tt[kHistItems];
    uint32_t key[kHistItems];
#pragma unroll
    for (int k = 0; k < kHistItems; ++k) {
      const int64_t idx = b * per_block + (int64_t)k * kThreads + threadIdx.x;  // coalesced
      tt[k] = idx < n ? tiles_touched[idx] : 0;
      key[k] = idx < n ? depth_keys[idx] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kHistItems; ++k) {
      const bool vis = tt[k] > 0;
      if (__ballot(vis) == 0) continue;  // a wave of culled records (neighbours are culled together)
      if (vis) {
        atomicAdd(&s_hist[0][key[k] & 255u], 1u);
        atomicAdd(&s_hist[1][(key[k] >> 8) & 255u], 1u);
      }
      match_add(vis, (key[k] >> 16) & 255u, s_hist[2]);
      top_add(vis, key[k] >> 24, s_hist[3]);
    }
  }
  __syncthreads();
  const int copy = (int)(blockIdx.x % kDepthHistCopies);
  uint32_t* h = copy == 0 ? hist : hist_extra + (int64_t)(copy - 1) * kDepthHistWords;
  for (int i = threadIdx.x; i < 4 * kRadix; i += kThreads) {
    const uint32_t c = (&s_hist[0][0])[i];
    if (c) atomicAdd(&h[i], c);
  }
}

// ---------------------------------------------------------------------------
// 3. pair emission
// ---------------------------------------------------------------------------
struct EmitArgs {
  const uint4* rec_words;        // records as 16-byte words, kRecordWords per record
  const uint32_t* sorted;        // visible records in depth order (emission in that order)
  const int32_t* tiles_touched;  // > 0: visible (emission in record order)
  int64_t* counts;
  int64_t cap, pair_cap;
  int tw_shift, th_shift;        // log2 of the tile shape (every supported shape is a power of two)
  int tiles_x, tiles_per_view;
  uint32_t* out_tiles;
  uint32_t* out_records;
  int passes, bits;              // tile digits and their width
  uint32_t* hist;                // tile-digit histograms, [passes][kTileDigits]
  uint32_t* hist_extra;
  uint64_t* status;              // look-back words
  uint32_t* tile_counter;
  uint32_t* big_rec;             // records with many tiles and their first pair: a wave's from the front,
  uint32_t* big_off;             // a work-group's from the back ([cap])
  uint32_t* big_count;           // of each kind
  const uint64_t* group_pairs;   // emission in record order: see ClearArgs (the tiles' pairs are in `status`)
  const uint32_t* group_visible;
};

// first tile id and extent in tiles (columns | rows << 16) of a record
struct TileRect {
  uint32_t first, extent;
  __device__ __forceinline__ uint32_t columns() const { return extent & 0xFFFFu; }
  __device__ __forceinline__ uint32_t tiles() const { return columns() * (extent >> 16); }
};
__device__ __forceinline__ TileRect tile_rect(const EmitArgs& a, const uint4& w0) {
  const uint32_t i0 = w0.z & 0xFFFFu, i1 = i0 + (w0.z >> 16);
  const uint32_t j0 = w0.w & 0xFFFFu, j1 = j0 + (w0.w >> 16);
  const uint32_t tx0 = i0 >> a.tw_shift, ty0 = j0 >> a.th_shift;
  const uint32_t ntx = (i1 >> a.tw_shift) - tx0 + 1u, nty = (j1 >> a.th_shift) - ty0 + 1u;
  return TileRect{w0.y * (uint32_t)a.tiles_per_view + ty0 * (uint32_t)a.tiles_x + tx0, ntx | (nty << 16)};
}

__device__ __forceinline__ void count_tile(const EmitArgs& a, uint32_t (*s_hist)[kTileDigits], uint32_t key) {
  const uint32_t mask = (1u << a.bits) - 1u;
  for (int p = 0; p < a.passes; ++p) atomicAdd(&s_hist[p][(key >> (a.bits * p)) & mask], 1u);
}

// One work-group tile of kThreads * ITEMS records, sorted ones or (BY_RECORD) all in index order: gather,
// scan, write.
template <int ITEMS, bool BY_RECORD>
__device__ __forceinline__ void emit_tile(const EmitArgs& a, int64_t n, int64_t t, int64_t ntiles,
                                          uint32_t (*s_hist)[kTileDigits], uint64_t* s_wave64, uint64_t* s_base) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  // item k of lane l is element k*64 + l of the wave's contiguous slice
  const int64_t base = t * kThreads * ITEMS + (int64_t)wid * 64 * ITEMS + lane;
  uint32_t rid[ITEMS], cnt[ITEMS];  // records and their tiles
  TileRect rect[ITEMS];
  uint64_t front = 0;  // the thread's share of the pairs in front of the tile
  if constexpr (BY_RECORD) {
    const int64_t per = emit_group_tiles(ntiles), g = t / per;
    for (int64_t i = threadIdx.x; i < g; i += kThreads) front += a.group_pairs[i];
    for (int64_t i = g * per + threadIdx.x; i < t; i += kThreads) front += a.status[i];
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int64_t at = base + k * 64;
    if constexpr (BY_RECORD) {
      rid[k] = (uint32_t)at;
      cnt[k] = (uint32_t)max(at < n ? a.tiles_touched[at] : 0, 0);
    } else {
      rid[k] = at < n ? a.sorted[at] : 0u;
    }
  }
  {
    uint4 w0[ITEMS];
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      const bool live = BY_RECORD ? cnt[k] > 0 : base + k * 64 < n;
      w0[k] = live ? a.rec_words[(size_t)kRecordWords * rid[k]] : make_uint4(0u, 0u, 0u, 0u);
    }
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      rect[k] = tile_rect(a, w0[k]);
      if constexpr (!BY_RECORD) cnt[k] = base + k * 64 < n ? rect[k].tiles() : 0u;
    }
  }
  // exclusive prefix of the tile counts in slice order; a count may pass 2^25 and 64 of them 2^31, so
  // the halves are scanned apart
  uint64_t off[ITEMS], run = 0;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t c = cnt[k];
    uint64_t inc = (uint32_t)wave_incl_scan((int)(c & 0xFFFFu));
    if (__ballot(c > 0xFFFFu)) inc += (uint64_t)(uint32_t)wave_incl_scan((int)(c >> 16)) << 16;
    off[k] = run + inc - c;
    run += ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(inc >> 32), 63) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)inc, 63);
  }
  if (lane == 0) s_wave64[wid] = run;
  __syncthreads();
  uint64_t before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    const uint64_t v = s_wave64[w];
    before += w < wid ? v : 0ull;
    total += v;
  }
  auto finish = [&](uint64_t ex) {  // the pairs up to the last tile
    a.counts[GS_COUNT_PAIRS] = (int64_t)(ex + total);
    if ((int64_t)(ex + total) > a.pair_cap) raise_flag(a.counts, GS_FLAG_PAIRS);
  };
  if constexpr (BY_RECORD) {
    __syncthreads();
    const uint64_t ex = group_sum(front, s_wave64);
    if (threadIdx.x == 0) *s_base = ex;
    if (t == ntiles - 1) {
      const int64_t per = emit_group_tiles(ntiles);
      uint64_t visible = 0;
      for (int64_t i = threadIdx.x; i * per < ntiles; i += kThreads) visible += a.group_visible[i];
      visible = group_sum(visible, s_wave64);
      if (threadIdx.x == 0) {
        finish(ex);
        a.counts[GS_COUNT_VISIBLE] = (int64_t)visible;
      }
    }
  } else if (wid == 0) {
    const uint64_t ex = lookback64_wave(a.status, t, total, a.counts);
    if (lane == 0) {
      *s_base = ex;
      if (t == ntiles - 1) finish(ex);
    }
  }
  __syncthreads();
  const uint64_t tile_base = *s_base + before;
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const TileRect r = rect[k];
    const uint32_t c = cnt[k];
    int64_t o = (int64_t)(tile_base + off[k]);
    const bool many = c > kBigFootprint;
    const bool huge = c > kHugeFootprint;
    const bool big = many && !huge && o < a.pair_cap;  // left to emit_big_kernel
    if (huge && o < a.pair_cap) {
      const uint32_t at = (uint32_t)a.cap - 1u - atomicAdd(a.big_count + 1, 1u);
      a.big_rec[at] = rid[k];
      a.big_off[at] = (uint32_t)o;
    }
    const uint64_t bm = __ballot(big);
    if (bm) {  // one device atomic for the wave's
      uint32_t at = 0;
      if (lane == __builtin_ctzll(bm)) at = atomicAdd(a.big_count, (uint32_t)__popcll(bm));
      at = (uint32_t)__builtin_amdgcn_readlane((int)at, __builtin_ctzll(bm)) + (uint32_t)lanemask_lt_count(bm);
      if (big) {
        a.big_rec[at] = rid[k];
        a.big_off[at] = (uint32_t)o;
      }
    }
    if (many) continue;
    uint32_t key = r.first, column = 0;
    for (uint32_t q = 0; q < c; ++q, ++o) {
      if (o < a.pair_cap) {
        a.out_tiles[o] = key;
        a.out_records[o] = rid[k];
        count_tile(a, s_hist, key);
      }
      const bool wrap = ++column == r.columns();
      key += wrap ? (uint32_t)a.tiles_x - r.columns() + 1u : 1u;
      column = wrap ? 0u : column;
    }
  }
}

// Depth first, the gather of one 16-byte word per visible record in depth order bounds it: a
// line of 128 B per record (437 MB for 4M records, 3.8 TB/s), ITEMS gathers of a
// thread in flight.  Scan and emission in one kernel write the rectangles and
// offsets nowhere: 4M records 117 us, where a depth pass that gathered and scanned
// (118 against 52 for a plain one) and the emission (33) took 99 more than the
// plain pass; what is won is the passes' uniform shape and three arrays.
// In record order it moves half of that (264 MB for the 5.7M records with these 4M among them) and no tile
// waits for another: the pairs in front of a tile are sums the zero fill has made of the tile counts.
// 75 us and 10 more in the zero fill, where claim and look-back of 2787 tiles took 113 (two tiles per claim
// make every look-back wait for a whole tile before: 18 ms); 32M records 309 and 53 against 434; 675K 18
// and 1 against 26.  (The histograms' adds are no part of it: counted by runs of equal tiles, the same.)
template <bool BY_RECORD>
__global__ void __launch_bounds__(kThreads) emit_kernel(EmitArgs a) {
  __shared__ uint32_t s_hist[kMaxTilePasses][kTileDigits];
  __shared__ uint64_t s_wave64[kThreads / 64], s_base;
  __shared__ uint32_t s_tile;
  const int64_t n_rec = count_clamped(a.counts, GS_COUNT_RECORDS, a.cap);
  const int64_t n = BY_RECORD ? n_rec : count_clamped(a.counts, GS_COUNT_VISIBLE, a.cap);
  const int items = emit_items(n_rec);
  const int64_t ntiles = (n + (int64_t)kThreads * items - 1) / ((int64_t)kThreads * items);
  if ((int64_t)blockIdx.x >= ntiles) return;
  for (int p = 0; p < a.passes; ++p)
    for (int i = threadIdx.x; i < kTileDigits; i += kThreads) s_hist[p][i] = 0u;
  for (int64_t t = blockIdx.x;; t += gridDim.x) {
    if constexpr (!BY_RECORD) {  // (a look-back waits for the tiles in front: taken in launch order)
      if (threadIdx.x == 0) s_tile = atomicAdd(a.tile_counter, 1u);
      __syncthreads();
      t = s_tile;
    }
    if (t >= ntiles) break;
    if (items == 1) emit_tile<1, BY_RECORD>(a, n, t, ntiles, s_hist, s_wave64, &s_base);
    else if (items == 4) emit_tile<4, BY_RECORD>(a, n, t, ntiles, s_hist, s_wave64, &s_base);
    else emit_tile<kEmitMaxItems, BY_RECORD>(a, n, t, ntiles, s_hist, s_wave64, &s_base);
    __syncthreads();
  }
  const int copy = (int)(blockIdx.x % kTileHistCopies);
  uint32_t* h = copy == 0 ? a.hist : a.hist_extra + (int64_t)(copy - 1) * kTileHistWords;
  for (int p = 0; p < a.passes; ++p)
    for (int i = threadIdx.x; i < kTileDigits; i += kThreads) {
      const uint32_t c = s_hist[p][i];
      if (c) atomicAdd(&h[p * kTileDigits + i], c);
    }
}

// Records whose footprint covers many tiles (a Gaussian close to the camera), written to the same slots
// (row-major tile order) the serial loop would use: a wave per record up to kHugeFootprint tiles, a
// work-group beyond.  2 x 70001 records of 37 tiles: 263 us with a work-group for every record.
template <bool BY_RECORD>
__device__ __forceinline__ void emit_footprint(const EmitArgs& a, uint32_t i, uint32_t first, uint32_t step,
                                               uint32_t (*s_hist)[kTileDigits]) {
  const uint32_t rid = a.big_rec[i];
  const TileRect r = tile_rect(a, a.rec_words[(size_t)kRecordWords * rid]);
  const int64_t o0 = a.big_off[i];
  const uint32_t c = BY_RECORD ? (uint32_t)a.tiles_touched[rid] : r.tiles();
  for (uint32_t q = first; q < c; q += step) {
    const int64_t o = o0 + q;
    if (o < a.pair_cap) {
      const uint32_t ty = q / r.columns(), tx = q % r.columns();
      const uint32_t key = r.first + ty * (uint32_t)a.tiles_x + tx;
      a.out_tiles[o] = key;
      a.out_records[o] = rid;
      count_tile(a, s_hist, key);
    }
  }
}
template <bool BY_RECORD>
__global__ void __launch_bounds__(kThreads) emit_big_kernel(EmitArgs a) {
  __shared__ uint32_t s_hist[kMaxTilePasses][kTileDigits];
  const uint32_t nbig = a.big_count[0], nhuge = a.big_count[1];
  // emit_kernel has finished (same stream): its partial histograms are final
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < a.passes * kTileDigits; i += kThreads) {
      uint32_t part[kTileHistCopies - 1];
#pragma unroll
      for (int c = 0; c < kTileHistCopies - 1; ++c) part[c] = a.hist_extra[c * kTileHistWords + i];
      uint32_t sum = 0;
#pragma unroll
      for (int c = 0; c < kTileHistCopies - 1; ++c) sum += part[c];
      if (sum) atomicAdd(&a.hist[i], sum);
    }
  }
  constexpr uint32_t kWaves = kThreads / 64;
  if (blockIdx.x * kWaves >= nbig && blockIdx.x >= nhuge) return;
  for (int p = 0; p < a.passes; ++p)
    for (int i = threadIdx.x; i < kTileDigits; i += kThreads) s_hist[p][i] = 0u;
  __syncthreads();
  for (uint32_t k = blockIdx.x * kWaves + (threadIdx.x >> 6); k < nbig; k += gridDim.x * kWaves)
    emit_footprint<BY_RECORD>(a, k, threadIdx.x & 63, 64, s_hist);
  for (uint32_t k = blockIdx.x; k < nhuge; k += gridDim.x)
    emit_footprint<BY_RECORD>(a, (uint32_t)a.cap - 1u - k, threadIdx.x, kThreads, s_hist);
  __syncthreads();
  for (int p = 0; p < a.passes; ++p)
    for (int i = threadIdx.x; i < kTileDigits; i += kThreads) {
      const uint32_t c = s_hist[p][i];
      if (c) atomicAdd(&a.hist[p * kTileDigits + i], c);
    }
}

// ---------------------------------------------------------------------------
// 5. tile ranges
// ---------------------------------------------------------------------------
// Four pairs a thread: 29M pairs 82 -> 30 us, 6.3M 15 -> 8.
__global__ void ranges_kernel(const uint32_t* __restrict__ tiles, const int64_t* counts, int64_t pair_cap,
                              int64_t n_tile_ids, uint32_t* __restrict__ ranges) {
  const int64_t m = count_clamped(counts, GS_COUNT_PAIRS, pair_cap);
  const int lane = threadIdx.x & 63;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x * 4;
  // four pairs a thread (the array starts on a 256-byte boundary or is read word by word)
  const bool wide = ((uintptr_t)tiles & 15) == 0;
  for (int64_t j0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 4; j0 - 4 * lane < m; j0 += stride) {
    uint32_t k[6];
    if (wide && j0 + 4 <= m) {
      const uint4 v = *reinterpret_cast<const uint4*>(tiles + j0);
      k[1] = v.x, k[2] = v.y, k[3] = v.z, k[4] = v.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) k[i + 1] = j0 + i < m ? tiles[j0 + i] : 0xFFFFFFFFu;
    }
    k[0] = (uint32_t)__shfl_up((int)k[4], 1);
    k[5] = (uint32_t)__shfl_down((int)k[1], 1);
    if (lane == 0) k[0] = j0 > 0 ? tiles[j0 - 1] : 0xFFFFFFFFu;
    if (lane == 63) k[5] = j0 + 4 < m ? tiles[j0 + 4] : 0xFFFFFFFFu;
#pragma unroll
    for (int i = 1; i <= 4; ++i) {
      if ((int64_t)k[i] >= n_tile_ids) continue;  // past the end (never produced by emission)
      if (k[i - 1] != k[i]) ranges[2 * (int64_t)k[i]] = (uint32_t)(j0 + i - 1);
      if (k[i + 1] != k[i]) ranges[2 * (int64_t)k[i] + 1] = (uint32_t)(j0 + i);
    }
  }
}

// ---------------------------------------------------------------------------
// 7. work queue for the persistent tile kernels: tiles ordered by decreasing
//    list length, bucketed by floor(log2(length)) (empty tiles last); the order
//    inside a bucket is irrelevant because tiles are independent
// ---------------------------------------------------------------------------
constexpr int kQueueBins = 33;

__device__ __forceinline__ int queue_bin(const uint32_t* ranges, int64_t t) {
  const uint32_t len = ranges[2 * t + 1] - ranges[2 * t];
  return len == 0 ? 32 : __clz(len);  // 0 = longest (bit 31 set) ... 31 = length 1
}

__global__ void queue_hist_kernel(const uint32_t* __restrict__ ranges, int64_t n_tiles, uint32_t* __restrict__ qhist) {
  __shared__ uint32_t s_h[kQueueBins];
  for (int i = threadIdx.x; i < kQueueBins; i += blockDim.x) s_h[i] = 0u;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_tiles; t += stride)
    atomicAdd(&s_h[queue_bin(ranges, t)], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kQueueBins; i += blockDim.x)
    if (s_h[i]) atomicAdd(&qhist[i], s_h[i]);
}

// Each work-group ranks its tiles inside their bins with LDS atomics, then takes
// one range per non-empty bin from the global cursors: one global atomic per
// (work-group, bin) instead of one per tile (same-address atomics serialise).
__global__ void queue_scatter_kernel(const uint32_t* __restrict__ ranges, int64_t n_tiles,
                                     const uint32_t* __restrict__ qhist, uint32_t* __restrict__ qcur,
                                     uint32_t* __restrict__ queue) {
  __shared__ uint32_t s_base[kQueueBins];
  __shared__ uint32_t s_cnt[kQueueBins];
  __shared__ uint32_t s_off[kQueueBins];
  if (threadIdx.x == 0) {
    uint32_t acc = 0;
    for (int i = 0; i < kQueueBins; ++i) {
      s_base[i] = acc;
      acc += qhist[i];
    }
    if (blockIdx.x == 0) {
      queue[0] = 0u;  // head counters of the forward and backward tile kernels
      queue[1] = 0u;
    }
  }
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t0 = (int64_t)blockIdx.x * blockDim.x; t0 < n_tiles; t0 += stride) {
    for (int i = threadIdx.x; i < kQueueBins; i += blockDim.x) s_cnt[i] = 0u;
    __syncthreads();
    const int64_t t = t0 + threadIdx.x;
    const int bin = t < n_tiles ? queue_bin(ranges, t) : 0;
    const uint32_t rank = t < n_tiles ? atomicAdd(&s_cnt[bin], 1u) : 0u;
    __syncthreads();
    for (int i = threadIdx.x; i < kQueueBins; i += blockDim.x)
      if (s_cnt[i]) s_off[i] = atomicAdd(&qcur[i], s_cnt[i]);
    __syncthreads();
    if (t < n_tiles) queue[2 + s_base[bin] + s_off[bin] + rank] = (uint32_t)t;
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// workspace layout
// ---------------------------------------------------------------------------
// counters [64], depth digit histograms [4][256], tile digit histograms, queue histogram and cursors
// [2][40], partial tile-digit histograms of emit_kernel [kTileHistCopies - 1], partial depth-digit
// histograms of depth_hist_kernel [kDepthHistCopies - 1][4][256]
constexpr int64_t kQueueWords = 2 * 40;
constexpr int64_t kTileHistAt = 64 + kDepthHistWords;
constexpr int64_t kQueueAt = kTileHistAt + kTileHistWords;
constexpr int64_t kTileExtraAt = kQueueAt + kQueueWords;
constexpr int64_t kDepthExtraAt = kTileExtraAt + (kTileHistCopies - 1) * kTileHistWords;
constexpr int64_t kFixedWords = kDepthExtraAt + (kDepthHistCopies - 1) * kDepthHistWords;
static_assert(kDepthExtraAt % 2 == 0 && 3 * kEmitGroups <= (kDepthHistCopies - 1) * kDepthHistWords, "the groups' sums fit");

struct SortWs {
  uint32_t* dkeys_a;     // [rc]
  uint32_t* dvals_a;     // [rc]
  uint32_t* dkeys_b;     // [rc]
  uint32_t* dvals_b;     // [rc]
  uint32_t* big_rec;     // [rc] visible records with large footprints
  uint32_t* big_off;     // [rc] their first pair
  uint32_t* ptiles_alt;  // [pc]
  uint32_t* precs_alt;   // [pc]
  uint32_t* fixed;       // see above
  uint32_t* dstatus;     // [radix tiles][4][256]
  uint64_t* estatus;     // [emission tiles]
  uint32_t* pstatus;     // [radix tiles][kTileHistWords]
  size_t bytes;
};

inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

SortWs sort_ws_layout(char* base, int64_t rc, int64_t pc) {
  SortWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off = align_up(off + bytes);
    return p;
  };
  w.dkeys_a = (uint32_t*)take(4 * (size_t)rc);
  w.dvals_a = (uint32_t*)take(4 * (size_t)rc);
  w.dkeys_b = (uint32_t*)take(4 * (size_t)rc);
  w.dvals_b = (uint32_t*)take(4 * (size_t)rc);
  w.big_rec = (uint32_t*)take(4 * (size_t)rc);
  w.big_off = (uint32_t*)take(4 * (size_t)rc);
  w.ptiles_alt = (uint32_t*)take(4 * (size_t)pc);
  w.precs_alt = (uint32_t*)take(4 * (size_t)pc);
  w.fixed = (uint32_t*)take(4 * (size_t)kFixedWords);
  w.dstatus = (uint32_t*)take(4 * (size_t)radix_tiles_bound(rc) * 4 * kRadix);
  w.estatus = (uint64_t*)take(8 * (size_t)emit_tiles_bound(rc));
  w.pstatus = (uint32_t*)take(4 * (size_t)radix_tiles_bound(pc) * kTileHistWords);
  w.bytes = off;
  return w;
}

// Order of work: by tile (emit in record order, group by tile, sort each list by depth) or depth first (sort
// the records, emit, group by tile).  By tile, the depth order costs a sort of every pair in its list, a few
// instructions per pair up to 1024 and more beyond; depth first, five passes over the records, each a few
// launch latencies at least.  Decided by what the host knows, the capacities (us of the whole binning, depth
// first -> by tile, capacity per record 2 if not said):
//   1M records, 1080p, 44 pairs a tile        145 ->  87     2.4M records, 352 a tile          200 -> 152
//   1M records, 320x180, 2290 a tile          116 -> 101     2M records, 160x90, 5446 a tile   136 -> 127
//   4096 records, 16 a record, 172 a tile      63 ->  42     4096 records, 98 a record         93 ->  73
//   20000 records, 91 a record, 514 a tile    136 -> 160     70001 records, 9 a record, 3204   103 -> 124
//   140002 records, 42 a record, 2641 a tile  250 -> 382
// Lists that are longer than their mean suggests are sorted all the same, linear in their length: 1M records in
// far views, the longest list 5532, 32862, 184409, 633173: 191 -> 185, 182 -> 187, 181 -> 258, 184 -> 259 (the frame's
// other kernels take 259, 563, 2537 and 24081).  Nearly all pairs in one list, 1M, 2M, 4M: 172 -> 217, 257 -> 342,
// 351 -> 649.
bool lists_by_tile(int64_t rc, int64_t pc, int64_t n_tile_ids) {
  const bool few = pc <= 4 * rc;
  return pc <= (few ? 4096 : 512) * n_tile_ids && (few || pc <= (int64_t)1 << 20);
}

int tile_bits(int64_t n_ids) {
  int b = 0;
  while (((int64_t)1 << b) < n_ids) ++b;
  return b;
}

}  // namespace

size_t bin_sort_ws_bytes(int64_t rc, int64_t pc) { return sort_ws_layout(nullptr, rc, pc).bytes; }

}  // namespace gs

extern "C" gs_status gs_bin_sort(const void* records, const uint32_t* depth_keys, const int32_t* tiles_touched,
                                 int32_t n_views, int32_t width, int32_t height, const gs_tuning* tuning,
                                 int64_t record_capacity, int64_t pair_capacity, uint32_t* pair_tiles,
                                 uint32_t* pair_records, uint32_t* tile_ranges, uint32_t* tile_queue,
                                 int64_t* counts, void* ws, size_t ws_bytes, void* stream) {
  using namespace gs;
  if (!records || !depth_keys || !tiles_touched || !tuning || !pair_tiles || !pair_records || !tile_ranges ||
      !counts || !ws)
    return GS_ERR_INVALID_ARG;
  if (n_views <= 0 || width <= 0 || height <= 0 || width > 65535 || height > 65535) return GS_ERR_INVALID_ARG;
  if (!tile_shape_supported(tuning->tile_w, tuning->tile_h)) return GS_ERR_UNSUPPORTED;
  if (record_capacity <= 0 || pair_capacity <= 0) return GS_ERR_INVALID_ARG;
  // look-back words carry 30-bit counts
  if (record_capacity >= ((int64_t)1 << 30) || pair_capacity >= ((int64_t)1 << 30)) return GS_ERR_INVALID_ARG;
  const SortWs w = sort_ws_layout((char*)ws, record_capacity, pair_capacity);
  if (ws_bytes < w.bytes) return GS_ERR_WORKSPACE;
  const int tw = tuning->tile_w, th = tuning->tile_h;
  const int tx_n = tiles_x(width, tw), ty_n = tiles_y(height, th);
  const int64_t tiles_per_view = (int64_t)tx_n * ty_n;
  const int64_t n_tile_ids = tiles_per_view * n_views;
  if (n_tile_ids >= ((int64_t)1 << 31)) return GS_ERR_INVALID_ARG;
  const int tbits = tile_bits(n_tile_ids);
  // tile digits of up to 9 bits, as few passes as that allows and of equal width
  const int tpasses = (tbits + 8) / 9;
  const int tdigit = tpasses ? (tbits + tpasses - 1) / tpasses : 0;
  hipStream_t s = (hipStream_t)stream;
  const dim3 blk(kThreads);
  auto grid_for = [](int64_t items) {
    int64_t g = (items + kThreads - 1) / kThreads;
    return dim3((unsigned)(g < 1 ? 1 : (g > 2048 ? 2048 : g)));
  };
  uint32_t* counters = w.fixed;
  uint32_t* dhist = w.fixed + 64;
  uint32_t* thist = w.fixed + kTileHistAt;
  uint32_t* dhist_extra = w.fixed + kDepthExtraAt;
  const int trb = tdigit == 9 ? 9 : 8;               // digit bits of the pass's instance (a word per value)
  const int64_t prow = (int64_t)tpasses << trb;  // look-back words of a radix tile over all tile passes
  const bool by_tile = lists_by_tile(record_capacity, pair_capacity, n_tile_ids);
  uint64_t* group_pairs = (uint64_t*)(w.fixed + kDepthExtraAt);
  uint32_t* group_visible = (uint32_t*)(group_pairs + kEmitGroups);
  // 0. zero the counters, histograms, look-back words and ranges; by tile: the emission tiles' sums
  {
    // (by tile, the partial depth histograms' words hold the groups' sums)
    const ClearArgs c{w.fixed, by_tile ? kDepthExtraAt : kFixedWords, w.dstatus, w.estatus, w.pstatus,
                      radix_tiles_bound(pair_capacity) * prow, tile_ranges, 2 * n_tile_ids,
                      tiles_touched, group_pairs, group_visible};
    const int64_t drt = by_tile ? 0 : radix_tiles_bound(record_capacity) * 4 * kRadix;
    const int64_t most = drt > c.pstatus_words ? drt : c.pstatus_words;
    dim3 grid = grid_for(most > kFixedWords ? most : kFixedWords);
    if (by_tile) {
      const int64_t tiles = emit_tiles_bound(record_capacity), groups = tiles < kEmitGroups ? tiles : kEmitGroups;
      if (grid.x < (unsigned)groups) grid.x = (unsigned)groups;
      hipLaunchKernelGGL(clear_front_kernel<true>, grid, blk, 0, s, c, counts, record_capacity);
    } else {
      hipLaunchKernelGGL(clear_front_kernel<false>, grid, blk, 0, s, c, counts, record_capacity);
    }
  }
  GS_LAUNCH_CHECK();
  const dim3 rblk(kRadixThreads);
  if (!by_tile) {
    // 1. histograms of the four depth digits
    hipLaunchKernelGGL(depth_hist_kernel, grid_for((record_capacity + kHistItems - 1) / kHistItems), blk, 0, s,
                       tiles_touched, depth_keys, record_capacity, counts, dhist, dhist_extra);
    GS_LAUNCH_CHECK();
    // 2. depth sort, 4 passes of 8 bits: selected records -> b -> a -> b -> a.  The first pass keeps
    //    the visible records (index order within a digit) and writes counts[GS_COUNT_VISIBLE].  Each
    //    pass adds the partial copies of its digit histogram.
    auto depth_pass = [&](int p, const uint32_t* kin, const uint32_t* vin, uint32_t* kout, uint32_t* vout) {
      return RadixPass{kin, vin, kout, vout, counts, p == 0 ? GS_COUNT_RECORDS : GS_COUNT_VISIBLE, GS_COUNT_RECORDS,
                       record_capacity, 8 * p, 8, dhist + p * kRadix, dhist_extra + p * kRadix,
                       kDepthHistCopies - 1, kDepthHistWords, w.dstatus + p * kRadix, (int64_t)4 * kRadix,
                       counters + 1 + p, counts, tiles_touched};
    };
    const dim3 dgrid = radix_grid(record_capacity);
    hipLaunchKernelGGL((radix_pass_kernel<8, true>), dgrid, rblk, 0, s,
                       depth_pass(0, depth_keys, nullptr, w.dkeys_b, w.dvals_b));
    hipLaunchKernelGGL((radix_pass_kernel<8, false>), dgrid, rblk, 0, s,
                       depth_pass(1, w.dkeys_b, w.dvals_b, w.dkeys_a, w.dvals_a));
    hipLaunchKernelGGL((radix_pass_kernel<8, false>), dgrid, rblk, 0, s,
                       depth_pass(2, w.dkeys_a, w.dvals_a, w.dkeys_b, w.dvals_b));
    hipLaunchKernelGGL((radix_pass_kernel<8, false>), dgrid, rblk, 0, s,
                       depth_pass(3, w.dkeys_b, w.dvals_b, w.dkeys_a, w.dvals_a));
    GS_LAUNCH_CHECK();
  }
  // 3. emission (+ tile-digit histograms), into the buffer from which the last tile pass ends in the
  //    caller's arrays
  EmitArgs e{};
  e.rec_words = (const uint4*)records;
  e.sorted = w.dvals_a;
  e.tiles_touched = tiles_touched;
  e.counts = counts;
  e.cap = record_capacity;
  e.pair_cap = pair_capacity;
  e.tw_shift = __builtin_ctz((unsigned)tw);
  e.th_shift = __builtin_ctz((unsigned)th);
  e.tiles_x = tx_n;
  e.tiles_per_view = (int)tiles_per_view;
  e.out_tiles = (tpasses % 2 == 0) ? pair_tiles : w.ptiles_alt;
  e.out_records = (tpasses % 2 == 0) ? pair_records : w.precs_alt;
  e.passes = tpasses;
  e.bits = tdigit;
  e.hist = thist;
  e.hist_extra = w.fixed + kTileExtraAt;
  e.status = w.estatus;
  e.tile_counter = counters + 24;
  e.big_rec = w.big_rec;
  e.big_off = w.big_off;
  e.big_count = counters + 32;  // two
  e.group_pairs = group_pairs;
  e.group_visible = group_visible;
  const int64_t eg = emit_tiles_bound(record_capacity);
  const dim3 egrid((unsigned)(eg < 2048 ? eg : 2048));
  if (by_tile) hipLaunchKernelGGL(emit_kernel<true>, egrid, blk, 0, s, e);
  else hipLaunchKernelGGL(emit_kernel<false>, egrid, blk, 0, s, e);
  if (by_tile) hipLaunchKernelGGL(emit_big_kernel<true>, dim3(512), blk, 0, s, e);
  else hipLaunchKernelGGL(emit_big_kernel<false>, dim3(512), blk, 0, s, e);
  GS_LAUNCH_CHECK();
  // 4. tile passes
  uint32_t* kin = e.out_tiles;
  uint32_t* vin = e.out_records;
  for (int p = 0; p < tpasses; ++p) {
    uint32_t* kout = (kin == pair_tiles) ? w.ptiles_alt : pair_tiles;
    uint32_t* vout = (vin == pair_records) ? w.precs_alt : pair_records;
    const RadixPass a{kin, vin, kout, vout, counts, GS_COUNT_PAIRS, GS_COUNT_PAIRS, pair_capacity, tdigit * p,
                      tdigit, thist + p * kTileDigits, nullptr, 0, 0,
                      w.pstatus + ((int64_t)p << trb), prow, counters + 16 + p, counts, nullptr};
    const dim3 pgrid = radix_grid(pair_capacity);
    if (trb == 9) hipLaunchKernelGGL((radix_pass_kernel<9, false>), pgrid, rblk, 0, s, a);
    else hipLaunchKernelGGL((radix_pass_kernel<8, false>), pgrid, rblk, 0, s, a);
    GS_LAUNCH_CHECK();
    kin = kout;
    vin = vout;
  }
  // 5. ranges
  hipLaunchKernelGGL(ranges_kernel, dim3(2048), blk, 0, s, pair_tiles, counts, pair_capacity, n_tile_ids,
                     tile_ranges);
  GS_LAUNCH_CHECK();
  // 6. depth order inside the lists
  if (by_tile) {
    // (the tile passes' look-back words are free by now: kTileHistWords for every 16384 pairs of capacity at least,
    // of which the chunks need two for every list of more than kListWave and for every 16384 pairs)
    static_assert(kTileHistWords * kListWave >= 4 * kListChunk, "room for the chunks");
    const ListArgs l{tile_ranges, depth_keys, pair_records, w.precs_alt, pair_tiles, w.ptiles_alt,
                     (uint2*)w.pstatus, counters + 40, (uint32_t)(radix_tiles_bound(pair_capacity) * kTileHistWords / 2),
                     n_tile_ids, (uint32_t)(record_capacity - 1)};
    const int64_t lg = (n_tile_ids + 3) / 4;
    hipLaunchKernelGGL(list_sort_kernel, dim3((unsigned)(lg < 65536 ? lg : 65536)), dim3(256), 0, s, l);
    if (pair_capacity > kListWave) hipLaunchKernelGGL(list_chunk_kernel, dim3(256), rblk, 0, s, l);
    int p = 0;
    for (int64_t run = kListChunk; run < pair_capacity; run *= kListFan)
      hipLaunchKernelGGL(list_merge_kernel, dim3(256), rblk, 0, s, l, p++);
    GS_LAUNCH_CHECK();
  }
  // 7. work queue
  if ((tuning->flags & GS_TUNE_WORK_QUEUE) && tile_queue) {
    uint32_t* qhist = w.fixed + kQueueAt;
    uint32_t* qcur = qhist + 40;
    hipLaunchKernelGGL(queue_hist_kernel, grid_for(n_tile_ids), blk, 0, s, tile_ranges, n_tile_ids, qhist);
    hipLaunchKernelGGL(queue_scatter_kernel, grid_for(n_tile_ids), blk, 0, s, tile_ranges, n_tile_ids, qhist, qcur,
                       tile_queue);
    GS_LAUNCH_CHECK();
  }
  return GS_OK;
}

// ---------------------------------------------------------------------------
// Variant of gs_bin_sort for callers that cannot allocate: its workspace is a
// file-scope device array.  Host code only ever uses the address that
// hipGetSymbolAddress reports for the current device (the array's own name is
// a host-side stand-in, not a device address).
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[GS_STATIC_SCRATCH_BYTES];

namespace gs {
namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's copy of `scratch`, looked up once per device.
gs_status static_scratch(void** out) {
  int dev = -1;
  GS_HIP_CHECK(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return GS_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    GS_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return GS_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return GS_OK;
}

}  // namespace
}  // namespace gs

extern "C" gs_status gs_bin_sort_static(const void* records, const uint32_t* depth_keys,
                                        const int32_t* tiles_touched, int32_t n_views, int32_t width, int32_t height,
                                        const gs_tuning* tuning, int64_t record_capacity, int64_t pair_capacity,
                                        uint32_t* pair_tiles, uint32_t* pair_records, uint32_t* tile_ranges,
                                        uint32_t* tile_queue, int64_t* counts, void* stream) {
  // the checks gs_bin_sort makes without a workspace come first, so a bad call
  // fails the same way before the scratch array is looked up
  if (!records || !depth_keys || !tiles_touched || !tuning || !pair_tiles || !pair_records || !tile_ranges ||
      !counts)
    return GS_ERR_INVALID_ARG;
  if (record_capacity <= 0 || pair_capacity <= 0) return GS_ERR_INVALID_ARG;
  if (record_capacity >= ((int64_t)1 << 30) || pair_capacity >= ((int64_t)1 << 30)) return GS_ERR_INVALID_ARG;
  if (gs::bin_sort_ws_bytes(record_capacity, pair_capacity) > (size_t)GS_STATIC_SCRATCH_BYTES)
    return GS_ERR_SCRATCH;
  void* ws = nullptr;
  const gs_status st = gs::static_scratch(&ws);
  if (st != GS_OK) return st;
  return gs_bin_sort(records, depth_keys, tiles_touched, n_views, width, height, tuning, record_capacity,
                     pair_capacity, pair_tiles, pair_records, tile_ranges, tile_queue, counts, ws,
                     (size_t)GS_STATIC_SCRATCH_BYTES, stream);
}
