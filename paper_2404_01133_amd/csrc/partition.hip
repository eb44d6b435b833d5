// Block partition of a Gaussian cloud (Sec. 3.2.2, Eq. 2): foreground
// normalisation, contraction of unbounded space into the cube (-2, 2)^3, a
// uniform grid over the contracted x and y, and the Gaussians grouped by
// block with their original order kept inside a block.
//
// Stages (all sizes known on the host, nothing synchronises):
//   1. z range of all centres (order-preserving integer min / max)
//   2. per centre: block id in FP64 (fixed operation order; this file is
//      compiled with -ffp-contract=off), (id, index) pairs, digit histograms
//   3. one or two stable 8-bit radix passes by block id (the binning's pass)
//   4. block offsets from the boundaries of the sorted ids
// plus a gather of all attribute arrays into the new order.
#include "radix.h"

namespace gs {
namespace {

struct PartArgs {
  const float* means;  // [3][n]
  int64_t n;
  double xlo, xhi, ylo, yhi;  // foreground x / y extent (lo < hi)
  const uint32_t* zr;         // device: order-mapped z min, z max
  int32_t nx, ny;
};

// float bits -> unsigned integer with the same order (and back)
__device__ __forceinline__ uint32_t order_key(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float order_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

__global__ void part_clear_kernel(uint32_t* __restrict__ words, int64_t n_words, int64_t* __restrict__ counts,
                                  int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_words; i += stride) words[i] = 0u;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    words[0] = 0xFFFFFFFFu;  // z min (order-mapped), shrinks
    words[1] = 0u;           // z max (order-mapped), grows
    for (int k = 0; k < GS_COUNT_SLOTS; ++k) counts[k] = 0;
    counts[GS_COUNT_RECORDS] = n;
  }
}

__global__ void __launch_bounds__(256) zrange_kernel(const float* __restrict__ z, int64_t n, uint32_t* __restrict__ zr) {
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
#pragma unroll 4
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint32_t k = order_key(z[i]);
    lo = k < lo ? k : lo;
    hi = k > hi ? k : hi;
  }
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t a = __shfl_xor(lo, off, 64), b = __shfl_xor(hi, off, 64);
    lo = a < lo ? a : lo;
    hi = b > hi ? b : hi;
  }
  // one atomic pair per work-group: on one address they take 11.5 ns each, one after the other
  // (one per wave: 101 us for 5M Gaussians)
  __shared__ uint32_t s_lo[4], s_hi[4];
  if ((threadIdx.x & 63) == 0) {
    s_lo[threadIdx.x >> 6] = lo;
    s_hi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      lo = s_lo[w] < lo ? s_lo[w] : lo;
      hi = s_hi[w] > hi ? s_hi[w] : hi;
    }
    atomicMin(&zr[0], lo);
    atomicMax(&zr[1], hi);
  }
}

// index of the grid cell along one axis: the number of interior boundaries
// -2 + 4k/cells (k = 1 .. cells-1) that are <= c; a NaN coordinate gets 0
__device__ __forceinline__ int grid_index(double c, int cells) {
  if (!(c == c)) return 0;
  double e = (c + 2.0) * (double)cells * 0.25;  // estimate, corrected exactly below
  int k = e < 0.0 ? 0 : (e > (double)(cells - 1) ? cells - 1 : (int)e);
  while (k + 1 <= cells - 1 && (-2.0 + (4.0 * (double)(k + 1)) / (double)cells) <= c) ++k;
  while (k >= 1 && (-2.0 + (4.0 * (double)k) / (double)cells) > c) --k;
  return k;
}

__device__ __forceinline__ uint32_t block_of(const PartArgs& a, double zlo, double zhi, double x, double y,
                                             double z) {
  const double q0 = (2.0 * (x - a.xlo)) / (a.xhi - a.xlo) - 1.0;
  const double q1 = (2.0 * (y - a.ylo)) / (a.yhi - a.ylo) - 1.0;
  const double q2 = (2.0 * (z - zlo)) / (zhi - zlo) - 1.0;
  const double m0 = fabs(q0), m1 = fabs(q1), m2 = fabs(q2);
  const bool nan = !(m0 == m0) || !(m1 == m1) || !(m2 == m2);
  double nrm = m0 > m1 ? m0 : m1;
  nrm = m2 > nrm ? m2 : nrm;
  double c0 = q0, c1 = q1;
  if (!nan && nrm > 1.0) {  // Eq. 2, outer region
    const double s = 2.0 - 1.0 / nrm;
    c0 = s * (q0 / nrm);
    c1 = s * (q1 / nrm);
  }
  return (uint32_t)(grid_index(c1, a.ny) * a.nx + grid_index(c0, a.nx));
}

__global__ void __launch_bounds__(kThreads) part_ids_kernel(PartArgs a, uint32_t* __restrict__ keys,
                                                            uint32_t* __restrict__ vals,
                                                            uint32_t* __restrict__ block_id, int passes,
                                                            uint32_t* __restrict__ hist) {
  __shared__ uint32_t s_hist[2][kRadix];
  for (int k = threadIdx.x; k < 2 * kRadix; k += kThreads) (&s_hist[0][0])[k] = 0u;
  __syncthreads();
  const double zlo = (double)order_value(a.zr[0]), zhi = (double)order_value(a.zr[1]);
  const int64_t n = a.n;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint32_t b = block_of(a, zlo, zhi, (double)a.means[i], (double)a.means[n + i], (double)a.means[2 * n + i]);
    keys[i] = b;
    vals[i] = (uint32_t)i;
    if (block_id) block_id[i] = b;
    atomicAdd(&s_hist[0][b & 255u], 1u);
    if (passes > 1) atomicAdd(&s_hist[1][(b >> 8) & 255u], 1u);
  }
  __syncthreads();
  for (int k = threadIdx.x; k < passes * kRadix; k += kThreads) {
    const uint32_t c = (&s_hist[0][0])[k];
    if (c) atomicAdd(&hist[k], c);
  }
}

// block_off[b] = first position of the sorted ids holding an id >= b
__global__ void part_offsets_kernel(const uint32_t* __restrict__ ids, int64_t n, int32_t n_blocks,
                                    int64_t* __restrict__ block_off) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
    const int64_t cur = ids[j];
    const int64_t prev = j == 0 ? -1 : (int64_t)ids[j - 1];
    for (int64_t b = prev + 1; b <= cur; ++b) block_off[b] = j;
    if (j == n - 1)
      for (int64_t b = cur + 1; b <= n_blocks; ++b) block_off[b] = n;
  }
}

__global__ void part_empty_kernel(int64_t* __restrict__ block_off, int32_t n_blocks) {
  for (int b = threadIdx.x; b <= n_blocks; b += blockDim.x) block_off[b] = 0;
}

// cells of the grid in contracted coordinates (x0, x1, y0, y1): the boundaries
// grid_index compares against, outermost ends open, so a point's cell is its block
__global__ void part_cells_kernel(int32_t nx, int32_t ny, double* __restrict__ cells) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nx * ny) return;
  const int ix = b % nx, iy = b / nx;
  const double inf = __builtin_inf();
  double* c = cells + 4 * (int64_t)b;
  c[0] = ix == 0 ? -inf : -2.0 + (4.0 * (double)ix) / (double)nx;
  c[1] = ix == nx - 1 ? inf : -2.0 + (4.0 * (double)(ix + 1)) / (double)nx;
  c[2] = iy == 0 ? -inf : -2.0 + (4.0 * (double)iy) / (double)ny;
  c[3] = iy == ny - 1 ? inf : -2.0 + (4.0 * (double)(iy + 1)) / (double)ny;
}

// ---------------------------------------------------------------------------
// dst[c][k] = src[c][perm[k]] for every component plane of a Gaussian set.
//
// A block's Gaussians lie all over an unordered source, in ascending order: a
// 128-byte line of a source plane holds Gaussians of as many blocks as it has
// words, and read block after block it is fetched once for each.  So the
// destination is cut into tiles of one wave's width and the tiles are taken by
// their first source index: the tiles of different blocks that read the same
// stretch of the source are taken by one work-group and its neighbours, on one XCD
// (work-groups go round-robin to the eight, so XCD x gets the x-th eighth of the
// order).  The order is a counting sort into kGatherBuckets stretches, kept with
// its counters in the last destination plane, whose first tiles are gathered at
// the end.  Any permutation is right; one without such runs gains nothing.
// Measured, 5M Gaussians in 36 blocks (59 planes, 2.36 GB to move): in natural
// order 4.06 ms; ordered by tiles of 256 to 1024 with a tile per work-group 1.15 ms,
// whatever the tile and the planes per launch row (each 4-byte load filled a line
// of its CU's cache: 38 GB from L2); with groups of tiles see gather_kernel.
// ---------------------------------------------------------------------------
constexpr int kGatherTile = 64;
constexpr int kGatherThreads = 512;
constexpr int kGatherPerWave = 8;                    // tiles of a wave
constexpr int kGatherGroup = kGatherThreads / 64 * kGatherPerWave;  // tiles of a work-group
constexpr int kGatherWindow = 8192;                  // source words of a plane staged in LDS
constexpr int kGatherBuckets = 16384;
constexpr int kGatherPlanes = 15;  // planes per launch row at most
constexpr int kXcds = 8;
// Below this the source planes stay in cache whatever the order, and the order's launches cost more than
// it wins: natural -> by stretches, 262144 Gaussians in random order 99 -> 150 us, in 36 blocks 81 -> 63; 700000
// 593 -> 481 and 435 -> 118 (already in order 98 -> 103)
constexpr int64_t kGatherOrdered = (int64_t)1 << 19;

struct GatherArgs {
  const float* src[5];
  float* dst[5];
  int comps[5];
  int64_t n_src, n;
  const uint32_t* perm;
  const uint32_t* order;  // tiles by first source index
  int64_t n_tiles;
  int planes, row;  // planes, planes per launch row

  __device__ __forceinline__ void plane(int c, const float*& s, float*& d) const {
    int a = 0;
    while (c >= comps[a]) c -= comps[a++];
    s = src[a] + (int64_t)c * n_src;
    d = dst[a] + (int64_t)c * n;
  }
};

// stretch of the source that holds the first index of tile t
__device__ __forceinline__ uint32_t gather_bucket(const uint32_t* __restrict__ perm, int64_t n_src, int64_t t) {
  const uint64_t b = (uint64_t)perm[t * kGatherTile] * kGatherBuckets / (uint64_t)n_src;
  return b < kGatherBuckets ? (uint32_t)b : (uint32_t)kGatherBuckets - 1u;
}

__global__ void gather_clear_kernel(uint32_t* __restrict__ at) { at[blockIdx.x * blockDim.x + threadIdx.x] = 0u; }

__global__ void gather_count_kernel(const uint32_t* __restrict__ perm, int64_t n_src, int64_t n_tiles,
                                    uint32_t* __restrict__ at) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_tiles) atomicAdd(&at[gather_bucket(perm, n_src, t)], 1u);
}

// counts -> first positions (one work-group)
__global__ void __launch_bounds__(1024) gather_scan_kernel(uint32_t* __restrict__ at) {
  __shared__ uint32_t s_wave[16];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  constexpr int kPer = kGatherBuckets / 1024;
  uint32_t c[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    c[i] = at[threadIdx.x * kPer + i];
    sum += c[i];
  }
  uint32_t run = (uint32_t)wave_incl_scan((int)sum);
  if (lane == 63) s_wave[wid] = run;
  __syncthreads();
  run -= sum;
  for (int w = 0; w < wid; ++w) run += s_wave[w];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    at[threadIdx.x * kPer + i] = run;
    run += c[i];
  }
}

__global__ void gather_place_kernel(const uint32_t* __restrict__ perm, int64_t n_src, int64_t n_tiles,
                                    uint32_t* __restrict__ at, uint32_t* __restrict__ order) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_tiles) order[atomicAdd(&at[gather_bucket(perm, n_src, t)], 1u)] = (uint32_t)t;
}

// tiles that the order and its counters cover in the last plane
__host__ __device__ constexpr int64_t gather_order_tiles(int64_t n_tiles) {
  return (n_tiles + kGatherBuckets + kGatherTile - 1) / kGatherTile;
}

// kGatherGroup tiles per work-group, a.row planes per launch row.  In the order above the tiles of a
// group read one stretch of the source, a few times the group's own length: it is staged in LDS by whole
// lines and gathered there; what lies beyond (tiles of sparse blocks, permutations without runs) is read from
// memory.  Read from memory one word per lane, each load took a cycle per lane in the CU's cache (64 lines):
// 861 us for 5M Gaussians in 36 blocks; from the window 565 (2.36 GB, 4.2 TB/s; with windows of 12288 and 16384
// words 600 and 668, 128 tiles a work-group 670, 32 tiles 711, 8 planes a row 586).
__global__ void __launch_bounds__(kGatherThreads) gather_kernel(GatherArgs a) {
  constexpr int kPer = kGatherWindow / kGatherThreads;
  __shared__ float s_win[kGatherWindow];
  __shared__ uint32_t s_lo, s_hi;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int64_t groups = (a.n_tiles + kGatherGroup - 1) / kGatherGroup;
  const int64_t eighth = (groups + kXcds - 1) / kXcds;
  const int64_t p = (int64_t)(blockIdx.x % kXcds) * eighth + blockIdx.x / kXcds;
  if (p >= groups) return;
  if (threadIdx.x == 0) {
    s_lo = 0xFFFFFFFFu;
    s_hi = 0u;
  }
  uint32_t tile[kGatherPerWave], idx[kGatherPerWave];  // (tile: the wave's)
  uint32_t live = 0;  // bit i: the lane has an element of tile i
#pragma unroll
  for (int i = 0; i < kGatherPerWave; ++i) {
    const int64_t q = p * kGatherGroup + i * (kGatherThreads / 64) + wid;  // neighbours in the order by different waves
    const uint32_t t = q >= a.n_tiles ? (uint32_t)a.n_tiles : a.order[q];
    tile[i] = (uint32_t)__builtin_amdgcn_readfirstlane((int)t);
    const int64_t k = (int64_t)tile[i] * kGatherTile + lane;
    idx[i] = k < a.n ? a.perm[k] : 0u;
    live |= (k < a.n ? 1u : 0u) << i;
  }
  __syncthreads();
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int i = 0; i < kGatherPerWave; ++i) lo = (live >> i & 1u) ? min(lo, idx[i]) : lo;
  atomicMin(&s_lo, lo);
  __syncthreads();
  lo = s_lo;
  uint32_t near = 0;  // bit i: element i is in the window
#pragma unroll
  for (int i = 0; i < kGatherPerWave; ++i) {
    const bool in = (live >> i & 1u) && idx[i] - lo < (uint32_t)kGatherWindow;
    near |= (in ? 1u : 0u) << i;
    hi = in ? max(hi, idx[i] - lo + 1u) : hi;
  }
  atomicMax(&s_hi, hi);
  __syncthreads();
  const int win = __builtin_amdgcn_readfirstlane((int)s_hi);  // words of the window in use
  const uint32_t far = live & ~near;
  const int p0 = (int)blockIdx.y * a.row;
  const int p1 = p0 + a.row < a.planes ? p0 + a.row : a.planes;
  for (int c = p0; c < p1; ++c) {
    const float* s;
    float* d;
    a.plane(c, s, d);
    if (win > 0) {
      const float* w = s + lo;
#pragma unroll
      for (int h = 0; h < kPer; h += 8) {
        if (h * kGatherThreads >= win) break;
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int j = (h + i) * kGatherThreads + (int)threadIdx.x;
          x[i] = j < win ? w[j] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) s_win[(h + i) * kGatherThreads + (int)threadIdx.x] = x[i];
      }
      __syncthreads();
    }
    float v[kGatherPerWave];
#pragma unroll
    for (int i = 0; i < kGatherPerWave; ++i) v[i] = s_win[near >> i & 1u ? idx[i] - lo : 0u];
    if (__ballot(far != 0u)) {
#pragma unroll
      for (int i = 0; i < kGatherPerWave; ++i)
        if (far >> i & 1u) v[i] = s[idx[i]];
    }
#pragma unroll
    for (int i = 0; i < kGatherPerWave; ++i)
      // (the tiles of the last plane that hold the order, which is still read, are gathered at the end)
      if ((live >> i & 1u) && (c < a.planes - 1 || tile[i] >= gather_order_tiles(a.n_tiles)))
        d[(int64_t)tile[i] * kGatherTile + lane] = v[i];
    __syncthreads();  // the window is rewritten
  }
}

// In natural order, a thread per element, a.row planes per launch row.
__global__ void __launch_bounds__(256) gather_plain_kernel(GatherArgs a) {
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k >= a.n) return;
  const uint32_t idx = a.perm[k];
  const int p0 = (int)blockIdx.y * a.row;
  const int p1 = p0 + a.row < a.planes ? p0 + a.row : a.planes;
  for (int c = p0; c < p1; ++c) {
    const float* s;
    float* d;
    a.plane(c, s, d);
    d[k] = s[idx];
  }
}

__global__ void __launch_bounds__(256) gather_rest_kernel(GatherArgs a) {
  const float* s;
  float* d;
  a.plane(a.planes - 1, s, d);
  const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (k < a.n && k < gather_order_tiles(a.n_tiles) * kGatherTile) d[k] = s[a.perm[k]];
}

struct PartWs {
  uint32_t* words;  // [0..1] z range, [2..7] tile counters, then hist [2][256]
  uint32_t* hist;
  uint32_t* status; // [2][ntiles][256]
  uint32_t* k0;
  uint32_t* v0;
  uint32_t* k1;
  uint32_t* v1;
  int64_t* counts;
  int64_t n_words;
  size_t bytes;
};

PartWs part_ws_layout(char* base, int64_t n) {
  PartWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* p = base ? base + off : nullptr;
    off += (bytes + 255) & ~(size_t)255;
    return p;
  };
  const int64_t ntiles = radix_tiles(n);
  w.n_words = 8 + 2 * kRadix + 2 * ntiles * kRadix;
  w.words = (uint32_t*)take(4 * (size_t)w.n_words);
  w.hist = w.words ? w.words + 8 : nullptr;
  w.status = w.words ? w.words + 8 + 2 * kRadix : nullptr;
  w.counts = (int64_t*)take(8 * GS_COUNT_SLOTS);
  w.k0 = (uint32_t*)take(4 * (size_t)n);
  w.v0 = (uint32_t*)take(4 * (size_t)n);
  w.k1 = (uint32_t*)take(4 * (size_t)n);
  w.v1 = (uint32_t*)take(4 * (size_t)n);
  w.bytes = off;
  return w;
}

unsigned grid_of(int64_t n, int64_t cap) {
  const int64_t g = (n + 255) / 256;
  return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace
}  // namespace gs

extern "C" size_t gs_partition_workspace_bytes(int64_t n) {
  if (n < 0) return 0;
  return gs::part_ws_layout(nullptr, n).bytes;
}

extern "C" gs_status gs_partition(const float* means, int64_t n, const double* xy_box, int32_t nx, int32_t ny,
                                  uint32_t* block_id, uint32_t* perm, int64_t* block_off, double* cells, void* ws,
                                  size_t ws_bytes, void* stream) {
  using namespace gs;
  if (!xy_box || !block_off || n < 0 || (n > 0 && (!means || !perm || !ws))) return GS_ERR_INVALID_ARG;
  if (n >= ((int64_t)1 << 32)) return GS_ERR_INVALID_ARG;
  if (nx <= 0 || ny <= 0 || (int64_t)nx * ny > 65536) return GS_ERR_INVALID_ARG;
  PartArgs a{};
  a.means = means;
  a.n = n;
  a.nx = nx;
  a.ny = ny;
  // ends of each printed interval in either order
  a.xlo = xy_box[0] < xy_box[2] ? xy_box[0] : xy_box[2];
  a.xhi = xy_box[0] < xy_box[2] ? xy_box[2] : xy_box[0];
  a.ylo = xy_box[1] < xy_box[3] ? xy_box[1] : xy_box[3];
  a.yhi = xy_box[1] < xy_box[3] ? xy_box[3] : xy_box[1];
  if (!(a.xhi > a.xlo) || !(a.yhi > a.ylo)) return GS_ERR_INVALID_ARG;
  const int32_t B = nx * ny;
  hipStream_t s = (hipStream_t)stream;
  if (cells) {
    hipLaunchKernelGGL(part_cells_kernel, dim3((B + 255) / 256), dim3(256), 0, s, nx, ny, cells);
    GS_LAUNCH_CHECK();
  }
  if (n == 0) {
    hipLaunchKernelGGL(part_empty_kernel, dim3(1), dim3(256), 0, s, block_off, B);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  if (ws_bytes < gs_partition_workspace_bytes(n)) return GS_ERR_WORKSPACE;
  PartWs w = part_ws_layout((char*)ws, n);
  a.zr = w.words;
  const int passes = B > kRadix ? 2 : 1;
  const int64_t ntiles = radix_tiles(n);
  hipLaunchKernelGGL(part_clear_kernel, dim3(grid_of(w.n_words, 2048)), dim3(256), 0, s, w.words, w.n_words,
                     w.counts, n);
  hipLaunchKernelGGL(zrange_kernel, dim3(grid_of(n, 512)), dim3(256), 0, s, means + 2 * n, n, w.words);
  hipLaunchKernelGGL(part_ids_kernel, dim3(grid_of(n, 1024)), dim3(kThreads), 0, s, a, w.k0, w.v0, block_id, passes,
                     w.hist);
  GS_LAUNCH_CHECK();
  const uint32_t* kin = w.k0;
  const uint32_t* vin = w.v0;
  for (int p = 0; p < passes; ++p) {
    const bool last = p == passes - 1;
    uint32_t* kout = (p % 2 == 0) ? w.k1 : w.k0;
    uint32_t* vout = last ? perm : ((p % 2 == 0) ? w.v1 : w.v0);
    const RadixPass ra{kin, vin, kout, vout, w.counts, GS_COUNT_RECORDS, GS_COUNT_RECORDS, n, 8 * p, 8,
                       w.hist + p * kRadix, nullptr, 0, 0, w.status + (int64_t)p * ntiles * kRadix, (int64_t)kRadix,
                       w.words + 2 + p, w.counts, nullptr};
    hipLaunchKernelGGL((radix_pass_kernel<8, false, true>), radix_grid(n), dim3(kRadixThreads), 0, s, ra);
    GS_LAUNCH_CHECK();
    kin = kout;
    vin = vout;
  }
  hipLaunchKernelGGL(part_offsets_kernel, dim3(grid_of(n, 4096)), dim3(256), 0, s, kin, n, B, block_off);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

extern "C" gs_status gs_gather_gaussians(const gs_gaussians* src, const uint32_t* perm, int64_t n,
                                         const gs_gaussian_grads* dst, void* stream) {
  using namespace gs;
  if (!src || !dst || n < 0 || (n > 0 && !perm)) return GS_ERR_INVALID_ARG;
  if (n == 0) return GS_OK;
  if (!src->means || !src->scales || !src->quats || !src->opac || !src->sh || !dst->means || !dst->scales ||
      !dst->quats || !dst->opac || !dst->sh)
    return GS_ERR_INVALID_ARG;
  if (src->attr_half != 0) return GS_ERR_UNSUPPORTED;
  if (src->sh_degree < 0 || src->sh_degree > 3) return GS_ERR_INVALID_ARG;
  const int planes = (src->sh_degree + 1) * (src->sh_degree + 1);
  hipStream_t s = (hipStream_t)stream;
  GatherArgs a{};
  const float* srcs[5] = {src->means, (const float*)src->scales, (const float*)src->quats, (const float*)src->opac,
                          (const float*)src->sh};
  float* dsts[5] = {dst->means, dst->scales, dst->quats, dst->opac, dst->sh};
  const int comps[5] = {3, 3, 4, 1, 3 * planes};
  for (int k = 0; k < 5; ++k) {
    a.src[k] = srcs[k];
    a.dst[k] = dsts[k];
    a.comps[k] = comps[k];
    a.planes += comps[k];
  }
  a.n_src = src->n;
  a.n = n;
  a.perm = perm;
  a.n_tiles = (n + kGatherTile - 1) / kGatherTile;
  if (n < kGatherOrdered || src->n <= 0) {
    a.row = 4;
    hipLaunchKernelGGL(gather_plain_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)((a.planes + 3) / 4)),
                       dim3(256), 0, s, a);
    GS_LAUNCH_CHECK();
    return GS_OK;
  }
  uint32_t* order = reinterpret_cast<uint32_t*>(dst->sh + (int64_t)(3 * planes - 1) * n);
  uint32_t* at = order + a.n_tiles;
  const dim3 tg((unsigned)((a.n_tiles + 255) / 256));
  hipLaunchKernelGGL(gather_clear_kernel, dim3(kGatherBuckets / 256), dim3(256), 0, s, at);
  hipLaunchKernelGGL(gather_count_kernel, tg, dim3(256), 0, s, perm, src->n, a.n_tiles, at);
  hipLaunchKernelGGL(gather_scan_kernel, dim3(1), dim3(1024), 0, s, at);
  hipLaunchKernelGGL(gather_place_kernel, tg, dim3(256), 0, s, perm, src->n, a.n_tiles, at, order);
  a.order = order;
  const int64_t groups = (a.n_tiles + kGatherGroup - 1) / kGatherGroup;
  const int64_t grid = (groups + kXcds - 1) / kXcds * kXcds;
  // planes per row: about 2048 work-groups at least
  const int64_t row = groups * a.planes / 2048;
  a.row = (int)(row < 2 ? 2 : row > kGatherPlanes ? kGatherPlanes : row);
  hipLaunchKernelGGL(gather_kernel, dim3((unsigned)grid, (unsigned)((a.planes + a.row - 1) / a.row)),
                     dim3(kGatherThreads), 0, s, a);
  const int64_t rest = gather_order_tiles(a.n_tiles) * kGatherTile;
  hipLaunchKernelGGL(gather_rest_kernel, dim3((unsigned)((rest + 255) / 256)), dim3(256), 0, s, a);
  GS_LAUNCH_CHECK();
  return GS_OK;
}
