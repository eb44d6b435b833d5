// Per-tile alpha compositing (Eq. 1 of the paper), forward.
//
// One work-group per (view, tile); one lane per pixel, each wave64 an 8x8
// pixel block of the tile (a 16x16 tile is four waves), cut into eight 4x2
// pixel groups of 8 lanes.  The tile's Gaussians are staged through LDS in
// batches (coalesced gathers of 48-byte records, one per lane); each group
// keeps its own depth-ordered list of the staged records whose footprint meets
// it, and the groups walk their lists side by side (a lane reads the record of
// its group), so a small footprint occupies one group's step rather than a
// whole wave's.  A lane is done when its transmittance would drop below 1e-4 (its
// x becomes NaN, on which every footprint test fails); a wave leaves when all its
// lanes are, the work-group when all waves have (block-wide vote before each batch).
//
// Compiled with -ffp-contract=off: alpha is computed by exactly the same
// operations as in the adjoint (explicit fmaf), so the backward's recomputed
// decisions match the forward's.
#include "tile.h"

namespace gs {
namespace {

// group shapes: the forward blends in 4x2 groups (eight per wave), the
// backward in 4x4 quadrants (its partial sums run over 16 lanes)
constexpr int kFwdGW = 4, kFwdGH = 2;
constexpr int kFwdGroups = 64 / (kFwdGW * kFwdGH);
static_assert(kFwdGroups == 8, "the forward uses wave_compact8");

template <int TW, int TH, int BATCH>
struct FwdLds {
  float4 w0[BATCH], w1[BATCH], w2[BATCH];
  float4 f[BATCH];  // footprint as floats: i0, j0, i1 - i0, j1 - j0
  alignas(16) uint8_t list[(TW * TH) / 64][kFwdGroups][kListStride<BATCH>];
  uint8_t cand[(TW * TH) / 64][BATCH];
  uint32_t odd;  // a record staged for the tile has a colour that is not finite
};

__device__ __forceinline__ bool colour_finite(float c) { return c <= 3.4028235e38f; }  // (colours are not negative)

// Colours that are not finite: times the weight 0 of an entry that is not used, or at a pixel that is done, they
// would make NaN of the sum.  They are staged as 0, and added to the pixels written that have used them, which
// is what the weighted sums come to.  Nothing of the walk is live here, not even the thread's index: a register
// more in it costs 1 to 3 %.  (Sixteen views of the block 1344 -> 1357 us, eight of the city 354 both; with the
// index kept 1371 and 358, as a second walk that selects 1450 and 414.)
template <int TW, int TH>
__device__ __forceinline__ void add_odd_colours(const TileArgs& ta, int tile_g, int wid, float* __restrict__ rgb,
                                                const int32_t* __restrict__ n_last) {
  uint32_t ones = ~0u;  // (unknown to the compiler: the lane is found again here and not kept)
  asm volatile("" : "+s"(ones));
  const int lane = (int)__builtin_amdgcn_mbcnt_hi(ones, __builtin_amdgcn_mbcnt_lo(ones, 0u));
  const int view = tile_g / ta.tiles_per_view, tile = tile_g - view * ta.tiles_per_view;
  const int tyi = tile / ta.tiles_x_n, txi = tile - tyi * ta.tiles_x_n;
  const LaneMap<TW, TH, kFwdGW, kFwdGH> m(txi, tyi, wid, lane);
  const bool inside = m.i < ta.W && m.j < ta.H;
  const int64_t plane = (int64_t)ta.H * ta.W, pix = (int64_t)m.j * ta.W + m.i;
  const int last = inside ? n_last[(int64_t)view * plane + pix] : 0;
  const uint32_t start = ta.ranges[2 * tile_g];
  float C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
  for (int k = 0; __ballot(k < last); ++k) {
    const float4* r = reinterpret_cast<const float4*>(&ta.records[ta.pair_records[start + (uint32_t)k]]);
    const float4 w2 = r[2];
    if (colour_finite(w2.x) & colour_finite(w2.y) & colour_finite(w2.z)) continue;
    const float4 w0 = r[0];
    Eval e;
    const bool in_fp = evaluate_f((float)m.i, (float)m.j, footprint_floats(w0), w0.x, w2.w, r[1], e);
    if ((k < last) & in_fp & (e.alpha >= kAlphaMin)) {
      C0 += colour_finite(w2.x) ? 0.0f : w2.x;
      C1 += colour_finite(w2.y) ? 0.0f : w2.y;
      C2 += colour_finite(w2.z) ? 0.0f : w2.z;
    }
  }
  if (inside) {
    float* out = rgb + (int64_t)view * 3 * plane + pix;
    out[0] += C0;
    out[plane] += C1;
    out[2 * plane] += C2;
  }
}

template <int TW, int TH, int BATCH>
__device__ __forceinline__ void raster_fwd_tile(const TileArgs& ta, FwdLds<TW, TH, BATCH>& lds, int tile_g,
                                                float bg0, float bg1, float bg2, float* __restrict__ rgb,
                                                float* __restrict__ T_final, int32_t* __restrict__ n_last) {
  constexpr int NT = TW * TH;
  const Record* __restrict__ records = ta.records;
  const uint32_t* __restrict__ pair_records = ta.pair_records;
  const uint32_t* __restrict__ ranges = ta.ranges;
  const int W = ta.W, H = ta.H, tiles_x_n = ta.tiles_x_n, tiles_per_view = ta.tiles_per_view;
  float4* s_w0 = lds.w0;
  float4* s_w1 = lds.w1;
  float4* s_w2 = lds.w2;
  float4* s_f = lds.f;
  const int view = tile_g / tiles_per_view;
  const int tile = tile_g - view * tiles_per_view;
  const int tyi = tile / tiles_x_n, txi = tile - tyi * tiles_x_n;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const LaneMap<TW, TH, kFwdGW, kFwdGH> qb(txi, tyi, wid);
  const int i = qb.i, j = qb.j;
  const bool inside = (i < W) && (j < H);
  // a pixel that is done has no x: every footprint test fails on it (a NaN's bits are above any float's)
  float fi = inside ? (float)i : __builtin_nanf("");
  const float fj = (float)j;
  const uint32_t start = ranges[2 * tile_g], end = ranges[2 * tile_g + 1];
  float T = 1.0f, C0 = 0.0f, C1 = 0.0f, C2 = 0.0f;
  int last = 0;
  uint8_t(*lists)[kListStride<BATCH>] = lds.list[wid];
  const uint8_t* my_list = lists[qb.g];
  if (threadIdx.x == 0) {
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    s_w0[BATCH - 1] = s_w1[BATCH - 1] = s_w2[BATCH - 1] = s_f[BATCH - 1] = zero;  // the null record
    lds.odd = 0u;
  }
  for (uint32_t b = start; b < end; b += BATCH - 1) {
    if (__syncthreads_and(!(fi == fi))) break;
    const int nb = (int)min((uint32_t)(BATCH - 1), end - b);
    for (int k = threadIdx.x; k < nb; k += NT) {
      const float4* r = reinterpret_cast<const float4*>(&records[pair_records[b + k]]);
      float4 a = r[0];
      const float4 w1 = r[1];
      a.y = q_limit(w1.w);
      s_w0[k] = a;
      s_w1[k] = w1;
      float4 w2 = r[2];
      // (colours are not negative: their bits grow with them, infinity and NaN above all)
      const uint32_t top = max(max(__float_as_uint(w2.x), __float_as_uint(w2.y)), __float_as_uint(w2.z));
      if (__builtin_expect(top >= 0x7F800000u, 0)) {  // added at the end
        w2.x = colour_finite(w2.x) ? w2.x : 0.0f;
        w2.y = colour_finite(w2.y) ? w2.y : 0.0f;
        w2.z = colour_finite(w2.z) ? w2.z : 0.0f;
        lds.odd = 1u;
      }
      s_w2[k] = w2;
      s_f[k] = footprint_floats(a);
    }
    clear_lists<BATCH, kFwdGroups>(lists);
    __syncthreads();
    int max_cnt = 0;
    if (__ballot(fi == fi))  // (a wave whose pixels are all done only stages)
      max_cnt = wave_compact8<BATCH>(s_w0, s_f, s_w1, s_w2, nb, qb.x0, qb.y0, lds.cand[wid], lists);
    const int base_idx = (int)(b - start);
    int last_k = -1;  // 16 x the batch index of the last entry used in this batch
    auto blend = [&](int k, float du, const float4& f, const float4& w1, const float4& w2) {
      Eval e;
      const bool in_fp = evaluate_f(fi, fj, f, du, w2.w, w1, e);
      bool use = in_fp & (e.alpha >= kAlphaMin);
      float alpha = use ? e.alpha : 0.0f;  // an entry that is not used leaves T and C as they are
      float Tn = T * (1.0f - alpha);
      const bool stop = Tn < kTMin;  // (T is not below it: only an entry in use takes it there)
      if (__ballot(stop)) {  // once per pixel
        alpha = stop ? 0.0f : alpha;
        Tn = stop ? T : Tn;
        use = use & !stop;
        fi = stop ? __builtin_nanf("") : fi;
      }
      const float aT = alpha * T;
      C0 = fmaf(w2.x, aT, C0);  // (colours are finite here)
      C1 = fmaf(w2.y, aT, C1);
      C2 = fmaf(w2.z, aT, C2);
      T = Tn;
      last_k = use ? k : last_k;
    };
    // four entries of the lane's group list per trip: one LDS read for the
    // four byte indices, all records' words in flight together (past the
    // group's count: the null record)
    for (int t = 0; t < max_cnt; t += 4) {
      // byte offsets (index * 16) of the four entries into the staged arrays
      const uint32_t pk = *reinterpret_cast<const uint32_t*>(&my_list[t]);
      // no pixel is left that is not done and has an entry (else: four null records)
      if (__ballot((fi == fi) & (pk != (uint32_t)(BATCH - 1) * 0x01010101u)) == 0) break;
      const uint32_t o0 = (pk & (BATCH - 1)) << 4, o1 = ((pk >> 8) & (BATCH - 1)) << 4;
      const uint32_t o2 = ((pk >> 16) & (BATCH - 1)) << 4, o3 = ((pk >> 24) & (BATCH - 1)) << 4;
      auto at = [](const float4* a, uint32_t o) {
        return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(a) + o);
      };
      auto at_x = [](const float4* a, uint32_t o) {
        return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(a) + o);
      };
      const float au = at_x(s_w0, o0), bu = at_x(s_w0, o1), cu = at_x(s_w0, o2), du = at_x(s_w0, o3);
      const float4 af = at(s_f, o0), a1 = at(s_w1, o0), a2 = at(s_w2, o0);
      const float4 bf = at(s_f, o1), b1 = at(s_w1, o1), b2 = at(s_w2, o1);
      const float4 cf = at(s_f, o2), c1 = at(s_w1, o2), c2 = at(s_w2, o2);
      const float4 df = at(s_f, o3), d1 = at(s_w1, o3), d2 = at(s_w2, o3);
      blend((int)o0, au, af, a1, a2);
      blend((int)o1, bu, bf, b1, b2);
      blend((int)o2, cu, cf, c1, c2);
      blend((int)o3, du, df, d1, d2);
    }
    if (last_k >= 0) last = base_idx + (last_k >> 4) + 1;
    __syncthreads();
  }
  if (inside) {
    const int64_t plane = (int64_t)H * W;
    const int64_t pix = (int64_t)j * W + i;
    float* out = rgb + (int64_t)view * 3 * plane + pix;
    out[0] = fmaf(T, bg0, C0);
    out[plane] = fmaf(T, bg1, C1);
    out[2 * plane] = fmaf(T, bg2, C2);
    T_final[(int64_t)view * plane + pix] = T;
    n_last[(int64_t)view * plane + pix] = last;
  }
  if (end > start && lds.odd) add_odd_colours<TW, TH>(ta, tile_g, wid, rgb, n_last);
}

// Bound by VALU issue (with the groups' lists, about 24 instructions and an
// exponential per entry).  Measured, us per call: eight 1600x900 views of the 20M
// city 384 before the lists left out unreachable groups, 374 with that, 337 with the
// loop free of per-entry count, done and stop selects; 16 views of a 2M block 1977,
// 1514, 1348, 1357 with colours tested; 4096 Gaussians at 256x256 53, 35, 30.  Six
// waves per SIMD for the multi-wave tiles (the compiler spills a dozen registers
// outside the loop): 1348 for the block, 1448 at five, 1440 at seven.
template <int TW, int TH, int BATCH>
__global__ void __launch_bounds__(TW* TH) __attribute__((amdgpu_waves_per_eu(TW * TH >= 128 ? 6 : 1))) raster_fwd_kernel(TileArgs ta, uint32_t* queue, float bg0, float bg1,
                                                            float bg2, float* __restrict__ rgb,
                                                            float* __restrict__ T_final,
                                                            int32_t* __restrict__ n_last) {
  __shared__ FwdLds<TW, TH, BATCH> lds;
  for_each_tile(ta, queue, 0, [&](int tile_g) {
    raster_fwd_tile<TW, TH, BATCH>(ta, lds, tile_g, bg0, bg1, bg2, rgb, T_final, n_last);
  });
}

template <int TW, int TH>
void launch_fwd(int batch, const TileArgs& ta, uint32_t* queue, hipStream_t s, const float* bg, float* rgb, float* T,
                int32_t* nl) {
  constexpr int NT = TW * TH;
  const dim3 grid = tile_grid(ta.n_tiles, queue != nullptr);
  if (batch == 64)
    hipLaunchKernelGGL((raster_fwd_kernel<TW, TH, 64>), grid, dim3(NT), 0, s, ta, queue, bg[0], bg[1], bg[2], rgb, T,
                       nl);
  else if (batch == 128)
    hipLaunchKernelGGL((raster_fwd_kernel<TW, TH, 128>), grid, dim3(NT), 0, s, ta, queue, bg[0], bg[1], bg[2], rgb,
                       T, nl);
  else
    hipLaunchKernelGGL((raster_fwd_kernel<TW, TH, 256>), grid, dim3(NT), 0, s, ta, queue, bg[0], bg[1], bg[2], rgb,
                       T, nl);
}

}  // namespace
}  // namespace gs

extern "C" gs_status gs_rasterize_fwd(const void* records, const uint32_t* pair_records, const uint32_t* tile_ranges,
                                      uint32_t* tile_queue, int32_t n_views, int32_t width, int32_t height,
                                      const float* bg,
                                      const gs_tuning* tuning, float* rgb, float* T_final, int32_t* n_last,
                                      void* stream) {
  using namespace gs;
  if (!records || !pair_records || !tile_ranges || !bg || !tuning || !rgb || !T_final || !n_last)
    return GS_ERR_INVALID_ARG;
  if (n_views <= 0 || width <= 0 || height <= 0 || width > 65535 || height > 65535) return GS_ERR_INVALID_ARG;
  const int tw = tuning->tile_w, th = tuning->tile_h;
  if (!tile_shape_supported(tw, th) || !batch_supported(tuning->batch)) return GS_ERR_UNSUPPORTED;
  const int tx = tiles_x(width, tw), ty = tiles_y(height, th);
  const int64_t tpv = (int64_t)tx * ty;
  const int64_t nblocks = tpv * n_views;
  if (nblocks >= ((int64_t)1 << 31)) return GS_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  const TileArgs ta{(const Record*)records, pair_records, tile_ranges, width, height, tx, (int)tpv, nblocks};
  uint32_t* q = ((tuning->flags & GS_TUNE_WORK_QUEUE) && tile_queue) ? tile_queue : nullptr;
  const int b = tuning->batch;
  if (tw == 16 && th == 16) launch_fwd<16, 16>(b, ta, q, s, bg, rgb, T_final, n_last);
  else if (tw == 8 && th == 8) launch_fwd<8, 8>(b, ta, q, s, bg, rgb, T_final, n_last);
  else if (tw == 16 && th == 8) launch_fwd<16, 8>(b, ta, q, s, bg, rgb, T_final, n_last);
  else if (tw == 32 && th == 8) launch_fwd<32, 8>(b, ta, q, s, bg, rgb, T_final, n_last);
  else launch_fwd<32, 16>(b, ta, q, s, bg, rgb, T_final, n_last);
  GS_LAUNCH_CHECK();
  return GS_OK;
}

