// Stable single-pass LSD radix pass (onesweep style), shared by the tile binning
// and the block partition.  Work-groups take tiles of keys from an atomic counter
// in launch order, rank their keys with wave64 ballot multisplit, publish
// per-digit tile counts and walk back over the predecessors' published counts
// (decoupled look-back), then scatter through LDS so the global writes of each
// digit run are contiguous.
//
// A work-group is 1024 threads with one tile in LDS (up to 16384 keys, 150 KB):
// one per CU.  What bounds a pass is the serial part of a tile and the look-back
// chain, not the bytes: 256-thread work-groups with 4096-key tiles took 12.7 us for
// a single tile (sixteen items ranked one after the other), and a pass over 4M keys
// had a chain of 980 tiles that all publish at about the same time.  Here a small
// input is cut into tiles of four items per thread, and a large one into tiles of
// sixteen, 245 for 4M keys, whose look-back reads 32 predecessors at a time.
// Mean per pass, us, before -> now: 4096 keys 12.7 -> 7.9; 0.5M to 0.8M keys
// 19.2 -> 15.9; 4M to 6.3M keys 52.5 -> 41.1; 12.6M 91 -> 76 (tiles of the old
// shape, ranking by 64-bit selects, against this).  Reading 64 predecessors at a
// time spilled registers (49 at 4M); a run-time item count made the loads of a
// thread wait for one another (66).
#pragma once

#include <type_traits>

#include "scan.h"

namespace gs {
namespace {

constexpr int kThreads = 256;
constexpr int kRadix = 256;
constexpr uint32_t kFlagAgg = 1u << 30;
constexpr uint32_t kFlagInc = 2u << 30;
constexpr uint32_t kValMask = (1u << 30) - 1;

constexpr int kRadixThreads = 1024;
constexpr int kRadixWaves = kRadixThreads / 64;
constexpr int kRadixMaxItems = 16;
constexpr int kRadixBlocks = 256;  // one work-group per CU (its LDS is nearly the CU's)
constexpr int kRadixMaxCopies = 7;  // partial histograms beside `hist`
constexpr int kLookWindow = 8;     // look-back words read per round by one thread

// Keys per thread of a pass over n keys: 4, 8, 12 or 16.  A small input spreads
// over the chip, up to 4M keys there is one tile per work-group; beyond that, as
// few rounds of tiles per work-group as their size allows, of equal size (6.3M
// keys: two rounds of twelve keys per thread, not one and a half of sixteen).
__host__ __device__ constexpr int radix_items(int64_t n) {
  const int64_t rows = (n + kRadixThreads - 1) / kRadixThreads;
  if (rows <= 128) return 4;
  if (rows <= 1024) return 8;
  if (rows <= (int64_t)kRadixBlocks * kRadixMaxItems) return kRadixMaxItems;
  const int64_t rounds = (rows + kRadixBlocks * kRadixMaxItems - 1) / (kRadixBlocks * kRadixMaxItems);
  return (int)((rows + 4 * kRadixBlocks * rounds - 1) / (4 * kRadixBlocks * rounds)) * 4;
}
__host__ __device__ constexpr int64_t radix_tiles(int64_t n) {
  const int64_t t = (int64_t)kRadixThreads * radix_items(n);
  return (n + t - 1) / t;
}
// upper bound of radix_tiles(m) over all m <= n
__host__ __device__ constexpr int64_t radix_tiles_bound(int64_t n) {
  const int64_t rows = (n + kRadixThreads - 1) / kRadixThreads;
  if (rows <= 128) return (rows + 3) / 4;
  if (rows <= 256) return 32;
  if (rows <= 1024) return (rows + 7) / 8;
  if (rows <= 2048) return 128;
  if (rows <= (int64_t)kRadixBlocks * kRadixMaxItems) return (rows + kRadixMaxItems - 1) / kRadixMaxItems;
  return (rows + kRadixBlocks * kRadixMaxItems - 1) / (kRadixBlocks * kRadixMaxItems) * kRadixBlocks;
}

// block-level exclusive scan of one u64 per thread (256 threads, 4 waves)
__device__ __forceinline__ uint64_t block_excl_scan64(uint64_t x, uint64_t* s_wave64, uint64_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  uint64_t inc = x;
  for (int off = 1; off < 64; off <<= 1) {
    const uint64_t y = __shfl_up(inc, off, 64);
    if (lane >= off) inc += y;
  }
  if (lane == 63) s_wave64[wid] = inc;
  __syncthreads();
  uint64_t wave_base = 0, tot = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    const uint64_t v = s_wave64[w];
    if (w < wid) wave_base += v;
    tot += v;
  }
  *total = tot;
  __syncthreads();
  return wave_base + inc - x;
}

// ---------------------------------------------------------------------------
// one stable LSD pass over a digit of up to RB bits; the digit histogram of the
// whole input was accumulated by the kernel that produced the keys
// ---------------------------------------------------------------------------
struct RadixPass {
  const uint32_t* keys_in;
  const uint32_t* vals_in;  // (unused by the compacting pass)
  uint32_t* keys_out;
  uint32_t* vals_out;
  const int64_t* counts_in;
  int count_idx;   // number of keys
  int size_idx;    // count whose value picks the tile size (the number of keys, or an upper bound
                   // of it for which the look-back words were cleared)
  int64_t cap;
  int shift, bits;              // digit = (key >> shift) & (2^bits - 1)
  const uint32_t* hist;         // digit histogram: `hist` plus
  const uint32_t* hist_extra;   // `hist_copies` (<= kRadixMaxCopies) partial copies, hist_stride words apart
  int hist_copies;
  int64_t hist_stride;
  uint32_t* status;             // look-back words, zeroed: [tile][status_stride >= 2^RB], one per digit
  int64_t status_stride;
  uint32_t* tile_counter;       // zeroed
  int64_t* counts;              // flags; the visible count (compacting pass)
  const int32_t* tiles_touched;  // compacting pass
};

template <int RB, int ITEMS = kRadixMaxItems>
struct RadixLds {
  static constexpr int kDigits = 1 << RB;
  static constexpr int kSegs = kRadixThreads / kDigits;  // look-back threads per digit
  static constexpr int kMaxTile = kRadixThreads * ITEMS;
  union {
    struct {
      uint32_t keys[kMaxTile], vals[kMaxTile];
    } s;
    struct {  // during the look-back, before the scatter
      uint32_t sum[kSegs][kDigits];
      uint32_t code[kSegs][kDigits];
      int32_t at[kDigits];
    } look;
    uint32_t words[2 * kMaxTile];  // (of those who sort a tile for themselves)
  } u;
  uint16_t wave_hist[kRadixWaves][kDigits];  // counts (at most 1024 keys of a wave), then positions in the tile
  uint32_t delta[kDigits];                   // output position less tile position of a digit
  uint32_t goff[kDigits];                    // keys of the whole input with a smaller digit
  uint32_t wave_tot[kRadixWaves];
  uint32_t tile;
};

// exclusive prefix over the digits, held by threads 0 .. kDigits - 1 (every thread calls it); total in *total
template <int RB, class Lds>
__device__ __forceinline__ uint32_t digit_excl_scan(Lds& lds, uint32_t x, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const uint32_t inc = (uint32_t)wave_incl_scan((int)x);
  if (lane == 63) lds.wave_tot[wid] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < (1 << RB) / 64; ++w) {
    const uint32_t s = lds.wave_tot[w];
    base += w < wid ? s : 0u;
    tot += s;
  }
  *total = tot;
  __syncthreads();
  return base + inc - x;
}

// Look-back of tile t over the published digit counts, all threads: kSegs
// threads per digit read kLookWindow words each per round (independent loads in
// flight), nearest predecessors first; the words are consumed in order up to the
// first inclusive prefix or the first one not published yet.  Positions before
// tile 0 read as an inclusive prefix of 0.  Returns the exclusive count to the
// threads of segment 0.
template <int RB>
__device__ __forceinline__ uint32_t radix_lookback(RadixLds<RB>& lds, const RadixPass& a, int64_t t) {
  using Lds = RadixLds<RB>;
  const int d = threadIdx.x & (Lds::kDigits - 1), seg = threadIdx.x >> RB;
  uint32_t excl = 0;
  bool open = seg == 0;  // segment 0 keeps the digit's state
  if (seg == 0) lds.u.look.at[d] = (int32_t)(t - 1);
  int64_t spins = 0;
  __syncthreads();
  for (;;) {
    const int at = lds.u.look.at[d];  // -2: done
    uint32_t sum = 0, used = 0, done = 0;
    if (at != -2) {
      uint32_t sv[kLookWindow];
      const int64_t k = (int64_t)at - seg * kLookWindow;
#pragma unroll
      for (int i = 0; i < kLookWindow; ++i)
        sv[i] = k - i >= 0 ? load_agent(a.status + (k - i) * a.status_stride + d) : kFlagInc;
      bool stop = false;
#pragma unroll
      for (int i = 0; i < kLookWindow; ++i) {
        const uint32_t flag = sv[i] & ~kValMask;
        stop |= flag == 0u;
        if (!stop && !done) {
          sum += sv[i] & kValMask;
          ++used;
          done = flag == kFlagInc;
        }
      }
      lds.u.look.sum[seg][d] = sum;
      lds.u.look.code[seg][d] = used | (done << 8);
    }
    __syncthreads();
    if (open) {
      int32_t next = at;
      bool stalled = false;
      for (int s = 0; s < Lds::kSegs; ++s) {
        const uint32_t c = lds.u.look.code[s][d];
        excl += lds.u.look.sum[s][d];
        next -= (int32_t)(c & 255u);
        if (c >> 8) {
          open = false;
          break;
        }
        if ((c & 255u) < (uint32_t)kLookWindow) {
          stalled = true;
          break;
        }
      }
      if (stalled && ++spins > kSpinLimit) {
        raise_flag(a.counts, GS_FLAG_WAIT);
        open = false;
      }
      lds.u.look.at[d] = open ? next : -2;
    }
    if (!__syncthreads_or(open)) return excl;
  }
}

// Lanes of `valid` whose digit equals the calling lane's (a wave's multisplit).
// Per bit one ballot m and the lane's bit as a mask s: lanes differ where m ^ s,
// a three-input boolean operation per 32 lanes.  (Written out with 32-bit masks:
// as 64-bit selects the compiler spent 13 VALU per bit instead of 4, and the
// ranking was most of a pass's time.)
template <int RB>
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t valid) {
  uint32_t lo = 0, hi = 0;  // lanes that differ
#pragma unroll
  for (int bit = 0; bit < RB; ++bit) {
    const int s = __builtin_amdgcn_sbfe((int)d, bit, 1);
    const uint64_t m = __ballot(s != 0);
    lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, (uint32_t)s, 0xF6);  // lo | (m ^ s)
    hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), (uint32_t)s, 0xF6);
  }
  return valid & ~(((uint64_t)hi << 32) | lo);
}

// Byte offset of element i of an array of words: 64 bits (WIDE), or 32, which beside a uniform base cost no
// address arithmetic, for arrays of fewer than 2^30 words.
template <bool WIDE>
__host__ __device__ constexpr std::conditional_t<WIDE, uint64_t, uint32_t> word_offset(uint32_t i) {
  return (std::conditional_t<WIDE, uint64_t, uint32_t>)i << 2;
}
static_assert(word_offset<true>(0xFFFFFFFFu) == 0x3FFFFFFFCull && word_offset<false>((1u << 30) - 1) == 0xFFFFFFFCu,
              "no offset wraps");
template <bool WIDE>
__device__ __forceinline__ uint32_t& word_at(uint32_t* p, uint32_t i) {
  return *reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(p) + word_offset<WIDE>(i));
}

template <int RB, int ITEMS, bool COMPACT, bool WIDE>
__device__ __forceinline__ void radix_tile(RadixLds<RB>& lds, const RadixPass& a, int64_t n, int64_t t) {
  using Lds = RadixLds<RB>;
  constexpr int kTileKeys = kRadixThreads * ITEMS;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t tile_base = t * kTileKeys;
  const uint32_t tile_n = (uint32_t)((n - tile_base) < kTileKeys ? (n - tile_base) : kTileKeys);
  const uint32_t* keys = a.keys_in + tile_base;
  const uint32_t* vals = COMPACT ? nullptr : a.vals_in + tile_base;
  const int32_t* tt = COMPACT ? a.tiles_touched + tile_base : nullptr;
  // wave w owns the contiguous slice [w*64*ITEMS, (w+1)*64*ITEMS) of the tile; item k of lane l is
  // element k*64 + l of that slice (coalesced loads)
  uint32_t key[ITEMS], val[ITEMS], rank[ITEMS];
  bool valid[ITEMS];
  const uint32_t slice = (uint32_t)(wid * 64 * ITEMS + lane);
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t li = slice + k * 64;
    const bool in_tile = li < tile_n;
    key[k] = in_tile ? keys[li] : 0u;
    if constexpr (COMPACT) {
      // (a culled record's key is read and dropped)
      valid[k] = (in_tile ? tt[li] : 0) > 0;
      val[k] = (uint32_t)tile_base + li;
    } else {
      valid[k] = in_tile;
      val[k] = in_tile ? vals[li] : 0u;
    }
  }
  auto digit = [&](uint32_t x) { return __builtin_amdgcn_ubfe(x, (uint32_t)a.shift, (uint32_t)a.bits); };
  // stable rank inside the wave: items in order k, lanes in order within an item
  uint16_t* hist = lds.wave_hist[wid];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint64_t vm = __ballot(valid[k]);
    if (vm == 0) {  // no valid item in the wave (a run of culled records, the end of the input)
      rank[k] = 0;
      continue;
    }
    const uint32_t d = digit(key[k]);
    const uint32_t prev = hist[d];
    const uint64_t peers = match_digit<RB>(d, vm);
    const uint32_t below = (uint32_t)lanemask_lt_count(peers);
    rank[k] = prev + below;
    if (valid[k] & (below == 0)) hist[d] = (uint16_t)(prev + (uint32_t)__popcll(peers));
    __builtin_amdgcn_wave_barrier();
  }
  __syncthreads();
  // per digit: count of the tile, published at once; prefix over the waves
  const int d = threadIdx.x & (Lds::kDigits - 1);
  uint32_t cnt = 0;
  uint32_t c[kRadixWaves];
  uint32_t* st = a.status + t * a.status_stride + d;
  if (threadIdx.x < Lds::kDigits) {
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) c[w] = lds.wave_hist[w][d];
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) {
      const uint32_t x = c[w];
      c[w] = cnt;
      cnt += x;
    }
    store_agent(st, (t == 0 ? kFlagInc : kFlagAgg) | cnt);
  }
  uint32_t tile_total;
  const uint32_t tile_excl = digit_excl_scan<RB>(lds, cnt, &tile_total);
  if (threadIdx.x < Lds::kDigits) {  // position of a wave's first key of the digit in the tile
#pragma unroll
    for (int w = 0; w < kRadixWaves; ++w) lds.wave_hist[w][d] = (uint16_t)(tile_excl + c[w]);
  }
  uint32_t excl = 0;
  if (t > 0) {
    excl = radix_lookback<RB>(lds, a, t);
    if (threadIdx.x < Lds::kDigits) store_agent(st, kFlagInc | (excl + cnt));
  }
  if (threadIdx.x < Lds::kDigits) lds.delta[d] = lds.goff[d] + excl - tile_excl;
  __syncthreads();  // (and the look-back's use of the key and value arrays is over)
  // local scatter by digit, then coalesced write-out
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (valid[k]) {
      const uint32_t pos = hist[digit(key[k])] + rank[k];
      lds.u.s.keys[pos] = key[k];
      lds.u.s.vals[pos] = val[k];
    }
  }
  __syncthreads();
  // (valid items only: tile_total = tile_n except in the compacting pass)
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const uint32_t i = (uint32_t)k * kRadixThreads + threadIdx.x;
    if (i < tile_total) {
      const uint32_t kk = lds.u.s.keys[i];
      const uint32_t out = lds.delta[digit(kk)] + i;
      word_at<WIDE>(a.vals_out, out) = lds.u.s.vals[i];
      word_at<WIDE>(a.keys_out, out) = kk;
    }
  }
}

// COMPACT: the least significant depth pass of the binning: reads every selected
// record's depth key, keeps those with tiles_touched > 0 (values = record index,
// in index order) and writes the visible count.  WIDE: 2^30 keys and more (the digits'
// counts stay below 2^30, what a look-back word holds).
template <int RB, bool COMPACT, bool WIDE = false>
__global__ void __launch_bounds__(kRadixThreads) radix_pass_kernel(RadixPass a) {
  using Lds = RadixLds<RB>;
  __shared__ Lds lds;
  const int64_t n = count_clamped(a.counts_in, a.count_idx, a.cap);
  const int items = radix_items(count_clamped(a.counts_in, a.size_idx, a.cap));
  const int64_t ntiles = (n + (int64_t)kRadixThreads * items - 1) / ((int64_t)kRadixThreads * items);
  if ((int64_t)blockIdx.x >= ntiles && !(COMPACT && blockIdx.x == 0)) return;
  uint32_t claimed = 0;  // (asked for before the histograms, and before a tile's end: it takes a round trip)
  if (threadIdx.x == 0) claimed = atomicAdd(a.tile_counter, 1u);
  // this digit's count over the whole input: `hist` plus the partial copies
  uint32_t hist_d = 0;
  if (threadIdx.x < Lds::kDigits && threadIdx.x < (1u << a.bits)) {
    hist_d = a.hist[threadIdx.x];
    uint32_t part[kRadixMaxCopies];
#pragma unroll
    for (int c = 0; c < kRadixMaxCopies; ++c) part[c] = c < a.hist_copies ? a.hist_extra[c * a.hist_stride + threadIdx.x] : 0u;
#pragma unroll
    for (int c = 0; c < kRadixMaxCopies; ++c) hist_d += part[c];
  }
  uint32_t total;
  const uint32_t goff = digit_excl_scan<RB>(lds, hist_d, &total);
  if (threadIdx.x < Lds::kDigits) lds.goff[threadIdx.x] = goff;
  if constexpr (COMPACT) {
    // the visible count = the digit histogram's total (taken by the later passes)
    if (blockIdx.x == 0 && threadIdx.x == 0) a.counts[GS_COUNT_VISIBLE] = (int64_t)total;
  }
  for (;;) {
    if (threadIdx.x == 0) lds.tile = claimed;
    for (int i = threadIdx.x; i < kRadixWaves * Lds::kDigits / 2; i += kRadixThreads)
      reinterpret_cast<uint32_t*>(&lds.wave_hist[0][0])[i] = 0u;
    __syncthreads();
    const int64_t t = lds.tile;
    if (t >= ntiles) break;
    if (items == 4) radix_tile<RB, 4, COMPACT, WIDE>(lds, a, n, t);
    else if (items == 8) radix_tile<RB, 8, COMPACT, WIDE>(lds, a, n, t);
    else if (items == 12) radix_tile<RB, 12, COMPACT, WIDE>(lds, a, n, t);
    else radix_tile<RB, kRadixMaxItems, COMPACT, WIDE>(lds, a, n, t);
    if (threadIdx.x == 0) claimed = atomicAdd(a.tile_counter, 1u);
    __syncthreads();
  }
}

inline dim3 radix_grid(int64_t cap) {
  const int64_t g = radix_tiles_bound(cap);
  return dim3((unsigned)(g < 1 ? 1 : (g > kRadixBlocks ? kRadixBlocks : g)));
}

}  // namespace
}  // namespace gs
