// Structural similarity between pairs of rendered images, the measure behind
// the data assignment of Eq. 3 (Sec. 3.2.2): SSIM of Wang et al. (2004) with
// an 11 x 11 Gaussian window of standard deviation 1.5 (normalised, zero
// padding outside the image), C1 = 0.01^2, C2 = 0.03^2, averaged over pixels
// and colour channels.
//
// One work-group per (32 x 32 output tile, image pair): both 42 x 42 input
// patches go to LDS, the horizontal pass writes the five windowed moments
// (x, y, x^2, y^2, xy) of 42 rows x 32 columns to LDS, the vertical pass
// finishes them per output pixel.  FP32 filtering; per-tile sums in FP64 are
// reduced per pair in a fixed order, so the result does not depend on
// scheduling.
//
// Bound by LDS and VALU issue and by the three channels' chain of load, row pass and
// column pass at three work-groups per CU.  A thread makes eight neighbouring outputs
// of a row, then four of a column, from one window it reads once (18 and 14 values for
// 88 and 44 taps; the products of the row pass once per value), the weights come with
// the launch, and the next channel's pixels are in flight during the passes.  13 pairs
// of 960 x 540: 170 us with one output at a time, 141 with the windows, 103 with the
// pixels ahead.
#include <cmath>

#include "gs_common.h"

namespace gs {
namespace {

constexpr int kSsimT = 32;               // output tile side
constexpr int kSsimR = 5;                // window radius
constexpr int kSsimP = kSsimT + 2 * kSsimR;  // patch side (42)
constexpr int kSsimThreads = 256;

constexpr int kSsimTaps = 2 * kSsimR + 1;
constexpr int kSsimRow = 8, kSsimCol = 4;  // outputs of a thread in the row and column pass
static_assert(kSsimT / kSsimCol * kSsimT == kSsimThreads, "one column run per thread");

struct SsimWindow {
  float w[kSsimTaps];
};
SsimWindow ssim_window() {
  SsimWindow out;
  double w[kSsimTaps], sum = 0.0;
  for (int k = -kSsimR; k <= kSsimR; ++k) {
    w[k + kSsimR] = std::exp(-(double)(k * k) / (2.0 * 1.5 * 1.5));
    sum += w[k + kSsimR];
  }
  for (int k = 0; k < kSsimTaps; ++k) out.w[k] = (float)(w[k] / sum);
  return out;
}

__global__ void __launch_bounds__(kSsimThreads) ssim_tile_kernel(const float* __restrict__ images, int64_t n_images,
                                                                 int W, int H, const int32_t* __restrict__ pairs,
                                                                 int tiles_x, SsimWindow win,
                                                                 double* __restrict__ partial) {
  __shared__ float s_x[kSsimP][kSsimP + 1];
  __shared__ float s_y[kSsimP][kSsimP + 1];
  __shared__ float s_h[5][kSsimP][kSsimT + 1];
  __shared__ double s_red[kSsimThreads / 64];
  const int tile = blockIdx.x, pair = blockIdx.y;
  const int ntiles = gridDim.x;
  const int tx0 = (tile % tiles_x) * kSsimT, ty0 = (tile / tiles_x) * kSsimT;
  const int64_t ia = pairs[2 * pair], ib = pairs[2 * pair + 1];
  const bool valid = ia >= 0 && ia < n_images && ib >= 0 && ib < n_images;
  const int64_t plane = (int64_t)H * W;
  double acc = 0.0;
  // the thread's share of the patches: pixel of each (-1: outside the image), values of the channel to come
  constexpr int kShare = (kSsimP * kSsimP + kSsimThreads - 1) / kSsimThreads;
  int64_t at[kShare];
  float px[kShare], py[kShare];
#pragma unroll
  for (int i = 0; i < kShare; ++i) {
    const int k = (int)threadIdx.x + i * kSsimThreads, r = k / kSsimP, q = k - r * kSsimP;
    const int gy = ty0 - kSsimR + r, gx = tx0 - kSsimR + q;
    at[i] = valid && r < kSsimP && gx >= 0 && gx < W && gy >= 0 && gy < H ? (int64_t)gy * W + gx : -1;
  }
  auto fetch = [&](int c) {
    const float* A = images + (ia * 3 + c) * plane;
    const float* B = images + (ib * 3 + c) * plane;
#pragma unroll
    for (int i = 0; i < kShare; ++i) {
      px[i] = at[i] >= 0 ? A[at[i]] : 0.0f;
      py[i] = at[i] >= 0 ? B[at[i]] : 0.0f;
    }
  };
  fetch(0);
  for (int c = 0; c < 3 && valid; ++c) {
    // (the row pass of the channel before is behind a barrier: the patches are free)
#pragma unroll
    for (int i = 0; i < kShare; ++i) {
      const int k = (int)threadIdx.x + i * kSsimThreads, r = k / kSsimP, q = k - r * kSsimP;
      if (r < kSsimP) {
        s_x[r][q] = px[i];
        s_y[r][q] = py[i];
      }
    }
    __syncthreads();
    if (c < 2) fetch(c + 1);  // in flight during the passes
    for (int k = threadIdx.x; k < kSsimP * (kSsimT / kSsimRow); k += kSsimThreads) {
      const int r = k / (kSsimT / kSsimRow), q = (k - r * (kSsimT / kSsimRow)) * kSsimRow;
      float m[kSsimRow][5] = {};
#pragma unroll
      for (int i = 0; i < kSsimRow + kSsimTaps - 1; ++i) {
        const float x = s_x[r][q + i], y = s_y[r][q + i];
        const float xx = x * x, yy = y * y, xy = x * y;
#pragma unroll
        for (int o = 0; o < kSsimRow; ++o) {
          const int t = i - o;
          if (t < 0 || t >= kSsimTaps) continue;
          m[o][0] = fmaf(win.w[t], x, m[o][0]);
          m[o][1] = fmaf(win.w[t], y, m[o][1]);
          m[o][2] = fmaf(win.w[t], xx, m[o][2]);
          m[o][3] = fmaf(win.w[t], yy, m[o][3]);
          m[o][4] = fmaf(win.w[t], xy, m[o][4]);
        }
      }
#pragma unroll
      for (int o = 0; o < kSsimRow; ++o)
#pragma unroll
        for (int u = 0; u < 5; ++u) s_h[u][r][q + o] = m[o][u];
    }
    __syncthreads();
    {
      const int r = (int)threadIdx.x / kSsimT * kSsimCol, q = (int)threadIdx.x % kSsimT;
      float m[kSsimCol][5] = {};
#pragma unroll
      for (int i = 0; i < kSsimCol + kSsimTaps - 1; ++i) {
#pragma unroll
        for (int u = 0; u < 5; ++u) {
          const float h = s_h[u][r + i][q];
#pragma unroll
          for (int o = 0; o < kSsimCol; ++o) {
            const int t = i - o;
            if (t >= 0 && t < kSsimTaps) m[o][u] = fmaf(win.w[t], h, m[o][u]);
          }
        }
      }
#pragma unroll
      for (int o = 0; o < kSsimCol; ++o) {
        if (tx0 + q >= W || ty0 + r + o >= H) continue;
        const float C1 = 0.01f * 0.01f, C2 = 0.03f * 0.03f;
        const float sxx = m[o][2] - m[o][0] * m[o][0], syy = m[o][3] - m[o][1] * m[o][1],
                    sxy = m[o][4] - m[o][0] * m[o][1];
        const float num = (2.0f * m[o][0] * m[o][1] + C1) * (2.0f * sxy + C2);
        const float den = (m[o][0] * m[o][0] + m[o][1] * m[o][1] + C1) * (sxx + syy + C2);
        acc += (double)(num / den);
      }
    }
  }
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kSsimThreads / 64; ++w) t += s_red[w];
    partial[(int64_t)pair * ntiles + tile] = valid ? t : __builtin_nan("");
  }
}

// per pair: tile sums in index order (fixed tree), divided by the sample count
__global__ void __launch_bounds__(256) ssim_reduce_kernel(const double* __restrict__ partial, int ntiles,
                                                          double count, float* __restrict__ out) {
  __shared__ double s[256];
  const int pair = blockIdx.x;
  double acc = 0.0;
  for (int t = threadIdx.x; t < ntiles; t += 256) acc += partial[(int64_t)pair * ntiles + t];
  s[threadIdx.x] = acc;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[pair] = (float)(s[0] / count);
}

}  // namespace
}  // namespace gs

extern "C" size_t gs_ssim_workspace_bytes(int32_t n_pairs, int32_t width, int32_t height) {
  using namespace gs;
  if (n_pairs <= 0 || width <= 0 || height <= 0) return 0;
  const int64_t tiles = (int64_t)((width + kSsimT - 1) / kSsimT) * ((height + kSsimT - 1) / kSsimT);
  return (size_t)(8 * tiles * n_pairs);
}

extern "C" gs_status gs_ssim(const float* images, int32_t n_images, int32_t width, int32_t height,
                             const int32_t* pairs, int32_t n_pairs, float* ssim, void* ws, size_t ws_bytes,
                             void* stream) {
  using namespace gs;
  if (!images || !pairs || !ssim || !ws || n_images <= 0 || n_pairs <= 0 || width <= 0 || height <= 0)
    return GS_ERR_INVALID_ARG;
  if (n_pairs > 65535) return GS_ERR_INVALID_ARG;
  if (ws_bytes < gs_ssim_workspace_bytes(n_pairs, width, height)) return GS_ERR_WORKSPACE;
  const int tiles_x = (width + kSsimT - 1) / kSsimT, tiles_y = (height + kSsimT - 1) / kSsimT;
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(ssim_tile_kernel, dim3(tiles_x * tiles_y, n_pairs), dim3(kSsimThreads), 0, s, images,
                     (int64_t)n_images, width, height, pairs, tiles_x, ssim_window(), (double*)ws);
  GS_LAUNCH_CHECK();
  hipLaunchKernelGGL(ssim_reduce_kernel, dim3(n_pairs), dim3(256), 0, s, (const double*)ws, tiles_x * tiles_y,
                     3.0 * (double)width * (double)height, ssim);
  GS_LAUNCH_CHECK();
  return GS_OK;
}
