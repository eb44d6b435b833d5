// Adjoint of the per-tile compositing (Sec. 3.1, differentiable rendering) and
// of the projection.
//
// Compositing adjoint: the forward's walk on 4x4 quadrants of 16 lanes, front
// to back, bounded by each pixel's n_last, with the blend state recomputed
// (colour in front is accumulated, colour behind = final colour - accumulated),
// so nothing per (pixel, Gaussian) is stored.  Per round a thread per staged
// record finds the quadrants it may reach; every (record, quadrant) hit owns a
// slot of nine sums in LDS, a record's slots side by side.  The nine partial
// gradients of a quadrant are summed with DPP row operations and stored to the
// slot (one plain LDS store for the wave's four quadrants), and the slots of a
// record are added in quadrant order and flushed with one FP32 atomic per (tile,
// Gaussian, quantity).  Then the projection adjoint chains each record's 2D
// partials back to the Gaussian's parameters.
//
// Why slots: the sums used to be added into one row per record with LDS float
// atomics, and those bounded the kernel (about 50 LDS cycles for the 36 lanes of a
// step, LDS busy 92 % of the time; a store takes two).  Now VALU issue bounds it: 76
// VALU and 5.5 LDS instructions per step of a wave, 21 of the VALU the reduction.
// Measured, 16 views of a 2M-Gaussian block at 1600x900: 5.16 ms with LDS atomics,
// 3.83 with slots and the moments below; 4096 Gaussians at 256x256 76 -> 66 us
// (one work-group per CU: the chain of steps); one 1M-Gaussian 1920x1080 view 102 ->
// 75 us.  Six waves per SIMD (a few spills outside the loop) against five: 3.88
// against 4.12 ms.
#include <type_traits>

#include "scan.h"
#include "tile.h"

namespace gs {
namespace {

// ---------------------------------------------------------------------------
// Sums of nine per-lane values over each 16-lane quadrant (a DPP row), all at
// once.  At each of four levels (partner lane ^ 15, ^ 7, ^ 3, ^ 1) two quantities
// share one register: lanes with bit 3 (2, 1, 0) clear keep the first, the others
// the second, and each lane adds the partner's copy of the quantity it keeps.
// Lanes l, l^15, l^7, l^8, ... of the four levels are the sixteen of the row, and
// a partner agrees in every bit already used, so it keeps the same quantities.
// The first two levels pick by banks of four lanes: two masked DPP adds write
// the two halves of one register, with no selects.  On return lane r of a row
// holds the row's total of value quad_value(r).  (Issue bound: 21 VALU and no LDS
// traffic; butterflies by selects and ds_swizzle took 27 and three LDS trips.)
// Every lane of the wave must be active.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}

__device__ __forceinline__ float quad_sum9(const float v[9], int lane) {
  float r0, r1, r2, r3, r4, s0, s1, s2;
  // a DPP source must have been written at least two instructions before
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %4, %16, %16 row_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %8, %8 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %0, %9, %9 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %1, %10, %10 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %1, %11, %11 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %12, %12 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %2, %13, %13 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %3, %14, %14 row_mirror row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %3, %15, %15 row_mirror row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %7, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %5, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %6, %2, %2 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %6, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "s_nop 1"
      : "=&v"(r0), "=&v"(r1), "=&v"(r2), "=&v"(r3), "=&v"(r4), "=&v"(s0), "=&v"(s1), "=&v"(s2)
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]), "v"(v[8]));
  const bool b1 = lane & 2, b0 = lane & 1;
  const float u0 = (b1 ? s1 : s0) + dpp_mov<0x1B>(b1 ? s0 : s1);  // quad_perm [3,2,1,0]
  const float u1 = s2 + dpp_mov<0x1B>(s2);
  return (b0 ? u1 : u0) + dpp_mov<0xB1>(b0 ? u0 : u1);  // quad_perm [1,0,3,2]
}

// value held by lane r of a row after quad_sum9, and whether the lane is the one that writes it
__device__ __forceinline__ int quad_value(int r) {
  return (r & 1) ? 8 : ((r & 2) << 1) | ((r & 4) >> 1) | ((r & 8) >> 3);
}
__device__ __forceinline__ bool quad_writes(int r) { return !(r & 1) || r == 1; }

// Partials per Gaussian: r, g, b, opacity, and with w = dL/dQ per pixel the sums
// of w p1, w p2, w p1^2, w p1 p2, w p2^2 (p = F d: the pixel's offset in the
// coordinates in which the Gaussian is round, Q = p1^2 + p2^2).  The second moments
// are taken of p and not of the offset d because dL/dSigma = -K (sum w d d^T) K
// with K ~ F^T F: for an elongated splat the moments of d cancel in it, those of p
// do not.  The sums over w leave out the factor -ln2 opac inside a tile
// (dG/dQ = -ln2 G); the flush applies it once.
constexpr int kG = 9;
constexpr int kGQ = 4;  // first partial with that factor
// Partial q of a staged record as it leaves the tile: second moments scaled, colour partials of a
// clamped channel (record colour exactly 0) dropped, so that the projection adjoint reads no records.
__device__ __forceinline__ float flush_value(uint32_t q, float v, const float4& w1, const float4& w2) {
  const float f = *(q < 3 ? &w2.x + q : &w1.w);  // the channel's colour or the opacity
  // (an infinite opacity is clamped at every pixel: its moments are 0 and stay 0)
  const float scaled = (q >= kGQ) & (v != 0.0f) ? v * (-0.69314718055994531f * f) : v;
  return (q < 3) & !(f > 0.0f) ? 0.0f : scaled;
}
// Words of the lists, which hold 16-bit entries (a type of its own kind: by the language's rules stores of
// entries and loads of uint32_t would be of different objects, which a compiler may reorder).
typedef uint32_t __attribute__((may_alias)) ListWord;
typedef uint32_t __attribute__((ext_vector_type(4), may_alias)) ListQuad;
constexpr int kBwdLdsOffsets = 1024;  // segment offsets staged in LDS by the view-major adjoint up to this many

// LDS of one tile.  Up to BATCH - 1 records are staged at a time (the last place is
// the null record) and walked in rounds of as many as have room for all their hits
// in the pool: small splats reach three to six of a 16x16 tile's sixteen
// quadrants, so about a hundred records share a round; splats that cover the tile
// take rounds of 25.  The pool is sized so that the six work-groups of a 16x16 tile
// that the kernel's registers allow fit a CU.
template <int TW, int TH, int BATCH>
struct BwdLds {
  static constexpr int kQuads = (TW * TH) / 16;
  static constexpr int kWaves = (TW * TH) / 64;
  static constexpr int kBatchBits = BATCH == 128 ? 7 : 6;
  static constexpr int kPool = kQuads * 25 < 511 ? kQuads * 25 : 511;  // + one slot for the null record
  static constexpr int kStride = BATCH + 2;  // list entries (u16); the odd dword count spreads the lists over banks
  static constexpr int kMaskBytes = kQuads <= 8 ? 1 : kQuads / 8;
  static_assert(BATCH == 64 || BATCH == 128, "records per round");
  static_assert(kPool >= kQuads, "a record always fits an empty pool");
  static_assert(((kPool + 1) << kBatchBits) <= 65536, "a list entry holds a record and a slot in 16 bits");
  static_assert(4 * kStride * 2 % 16 == 0, "whole 16-byte words");
  float4 w1[BATCH], w2[BATCH];
  float4 f[BATCH];  // footprint as floats: i0, j0, i1 - i0, j1 - j0
  alignas(16) float pool[((kPool + 1) * kG + 3) / 4 * 4];
  alignas(16) uint16_t list[kWaves][4][kStride];  // record | slot << kBatchBits
  float du[BATCH];
  uint32_t rec[BATCH];
  alignas(4) uint8_t mask[BATCH * kMaskBytes];  // quadrants a record may reach, bit wave * 4 + quadrant
  uint16_t end[BATCH];                          // hits of the staged records up to and with this one
  int quad_last[kQuads < 8 ? 8 : kQuads];  // entries that each quadrant must walk
  uint32_t odd;                            // a record staged for the tile has a colour that is not finite

  __device__ __forceinline__ uint32_t hits(int k) const {
    if constexpr (kMaskBytes == 1) return mask[k];
    else if constexpr (kMaskBytes == 2) return reinterpret_cast<const uint16_t*>(mask)[k];
    else return reinterpret_cast<const uint32_t*>(mask)[k];
  }
};

// Deterministic mode: per-(tile, record) partials are stored at slot
// base[record] + (the tile's row-major index within the record's footprint
// tiles), so a record's partials lie contiguous in ascending tile order and
// are summed in that order afterwards.
struct DetArgs {
  float* partial;        // [slots][kG]
  const uint32_t* base;  // [records]: first slot of each record
  int64_t slots;         // slots the workspace holds
};

template <int TW, int TH>
__device__ __forceinline__ int64_t det_slot(const DetArgs& d, uint32_t rid, int i0, int i1, int j0, int txi,
                                            int tyi) {
  const int tx0 = i0 / TW, ntx = i1 / TW - tx0 + 1, ty0 = j0 / TH;
  return (int64_t)d.base[rid] + (int64_t)(tyi - ty0) * ntx + (txi - tx0);
}

template <int TW, int TH, int BATCH, bool DET>
__device__ __forceinline__ void raster_bwd_tile(const TileArgs& ta, BwdLds<TW, TH, BATCH>& lds, int tile_g,
                                                const float* __restrict__ rgb, const float* __restrict__ T_final,
                                                const int32_t* __restrict__ n_last, const float* __restrict__ d_rgb,
                                                float* __restrict__ grad2d, const DetArgs& det) {
  using Lds = BwdLds<TW, TH, BATCH>;
  constexpr int NT = TW * TH;
  constexpr int KB = Lds::kBatchBits;
  const Record* __restrict__ records = ta.records;
  const uint32_t* __restrict__ pair_records = ta.pair_records;
  const uint32_t* __restrict__ ranges = ta.ranges;
  const int W = ta.W, H = ta.H, tiles_x_n = ta.tiles_x_n, tiles_per_view = ta.tiles_per_view;
  float4* s_w1 = lds.w1;
  float4* s_w2 = lds.w2;
  float4* s_f = lds.f;
  float* s_du = lds.du;
  uint32_t* s_rec = lds.rec;
  float* s_pool = lds.pool;
  const int view = tile_g / tiles_per_view;
  const int tile = tile_g - view * tiles_per_view;
  const int tyi = tile / tiles_x_n, txi = tile - tyi * tiles_x_n;
  const int lane = threadIdx.x & 63;
  const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const LaneMap<TW, TH, 4, 4> qb(txi, tyi, wid);
  const int i = qb.i, j = qb.j;
  const bool inside = (i < W) && (j < H);
  const uint32_t start = ranges[2 * tile_g];
  const int64_t plane = (int64_t)H * W;
  const int64_t pix = (int64_t)j * W + i;
  float g0 = 0.f, g1 = 0.f, g2 = 0.f, out0 = 0.f, out1 = 0.f, out2 = 0.f;
  int last = 0;
  if (inside) {
    const int64_t o = (int64_t)view * 3 * plane + pix;
    g0 = d_rgb[o];
    g1 = d_rgb[o + plane];
    g2 = d_rgb[o + 2 * plane];
    out0 = rgb[o];
    out1 = rgb[o + plane];
    out2 = rgb[o + 2 * plane];
    last = n_last[(int64_t)view * plane + pix];
  }
  // entries each quadrant / the tile must walk
  int ql = last;
  for (int off = 8; off > 0; off >>= 1) ql = max(ql, __shfl_xor(ql, off, 64));
  if ((lane & 15) == 0) lds.quad_last[threadIdx.x >> 4] = ql;
  if (threadIdx.x == 0) {
    const float4 zero = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    lds.odd = 0u;
    s_du[BATCH - 1] = 0.0f;
    s_f[BATCH - 1] = s_w1[BATCH - 1] = s_w2[BATCH - 1] = zero;
  }
  __syncthreads();
  int tile_last = 0;
  for (int q = 0; q < Lds::kQuads; ++q) tile_last = max(tile_last, lds.quad_last[q]);
  const float fi = (float)i, fj = (float)j;
  const int r = lane & 15;  // lane within the quadrant
  const bool writes = quad_writes(r);
  float* const my_pool = s_pool + quad_value(r);
  const uint16_t* my_list = lds.list[wid][qb.g];
  // transmittance and colour in front of the next entry, by the forward's own operations: the colour
  // behind (final colour less colour in front) then carries none of the roundings in front
  float T = 1.0f, A0 = 0.f, A1 = 0.f, A2 = 0.f;
  const uint32_t stop = start + (uint32_t)tile_last;
  for (uint32_t b = start; b < stop; b += BATCH - 1) {
    const int nb = (int)min((uint32_t)(BATCH - 1), stop - b);
    for (int k = threadIdx.x; k < nb; k += NT) {
      const uint32_t rid = pair_records[b + k];
      const float4* rp = reinterpret_cast<const float4*>(&records[rid]);
      const float4 w0 = rp[0];
      s_w1[k] = rp[1];
      s_w2[k] = rp[2];
      s_du[k] = w0.x;
      s_f[k] = footprint_floats(w0);
      s_rec[k] = rid;
    }
    __syncthreads();
    const int base_idx = (int)(b - start);
    // quadrants that walk each record and that it may reach, eight (two waves' blocks, 16x8 pixels) per thread
    for (int it = threadIdx.x; it < BATCH * Lds::kMaskBytes; it += NT) {
      const int k = it & (BATCH - 1), part = it >> KB;
      if (k >= nb) continue;
      const float4 w2 = s_w2[k];
      if (!((w2.x + w2.y) + w2.z <= 3.0e38f)) lds.odd = 1u;  // (colours are not negative)
      constexpr int kCols = TW >= 16 ? 4 : 2;
      const int x0 = txi * TW + (2 * part % (TW / 8)) * 8, y0 = tyi * TH + (2 * part / (TW / 8)) * 8;
      const float4 f = s_f[k], w1 = s_w1[k];
      GroupTest t;
      t.load<4, 4>(f, s_du[k], w2.w, w1, q_limit(w1.w), x0, y0);
      uint32_t m = 0;
#pragma unroll
      for (int ry = 0; ry < 2; ++ry) {
        const float r2 = t.row(4.0f * ry);
#pragma unroll
        for (int cx = 0; cx < kCols; ++cx) {
          const int g = (cx >> 1) * 4 + ry * 2 + (cx & 1);
          if (t.meets<4, 4>(4.0f * cx, 4.0f * ry) & t.reach(4.0f * cx, 4.0f * ry, r2) &
              (base_idx + k < lds.quad_last[part * 8 + g]))
            m |= 1u << g;
        }
      }
      lds.mask[k * Lds::kMaskBytes + part] = (uint8_t)m;
    }
    __syncthreads();
    const int my_last = last - base_idx;  // staged entries that the lane's pixel walks
    // slots by prefix sum over the records' hits (every wave for itself)
    int hit_end[BATCH / 64];
    uint32_t hits[BATCH / 64];
    {
      int carry = 0;
#pragma unroll
      for (int h = 0; h < BATCH / 64; ++h) {
        const int k = h * 64 + lane;
        hits[h] = k < nb ? lds.hits(k) : 0u;
        hit_end[h] = wave_incl_scan((int)__popc(hits[h])) + carry;
        carry = __builtin_amdgcn_readlane(hit_end[h], 63);
        if (wid == 0) lds.end[k] = (uint16_t)hit_end[h];
      }
    }
    // one entry of each quadrant's list: the four quadrants step (possibly
    // different) records side by side, each storing its sums to the hit's slot
    // (odd: see BwdLds)
    auto step = [&](auto odd, uint32_t k, uint32_t slot, float du, const float4& f, const float4& w1,
                    const float4& w2) {
      Eval e;
      const bool in_fp = evaluate_f(fi, fj, f, du, w2.w, w1, e);
      const bool use = ((int)k < my_last) & in_fp & (e.alpha >= kAlphaMin);
      // an entry that is not used leaves T and the colour in front as they are: a finite colour times 0
      // is 0, any other has to be left out
      const float alpha = use ? e.alpha : 0.0f;
      const float aT = alpha * T;
      A0 = fmaf(odd && !use ? 0.0f : w2.x, aT, A0);
      A1 = fmaf(odd && !use ? 0.0f : w2.y, aT, A1);
      A2 = fmaf(odd && !use ? 0.0f : w2.z, aT, A2);
      const float gc = fmaf(g0, w2.x, fmaf(g1, w2.y, g2 * w2.z));
      const float gb = fmaf(g0, out0 - A0, fmaf(g1, out1 - A1, g2 * (out2 - A2)));
      // hardware reciprocal (1 ulp): a correctly rounded division costs ~10 instructions
      // here and the gradient is not bit-compared
      const float one_a = 1.0f - alpha;
      const float inv1ma = __builtin_amdgcn_rcpf(one_a);
      // dL/dalpha = g . (colour T - (colour behind) / (1 - alpha))
      const float dalpha = fmaf(-gb, inv1ma, T * gc);
      const bool unclamped = use & (w1.w * e.G <= kAlphaMax);
      float c[kG];
      // (selected, not multiplied by 0: an unused entry adds nothing to its record even where the
      // loss gradient of the pixel is not finite)
      c[0] = use ? aT * g0 : 0.0f;
      c[1] = use ? aT * g1 : 0.0f;
      c[2] = use ? aT * g2 : 0.0f;
      c[3] = unclamped ? dalpha * e.G : 0.0f;
      c[4] = c[3] * e.p1;
      c[5] = c[3] * e.p2;
      c[6] = c[4] * e.p1;
      c[7] = c[4] * e.p2;
      c[8] = c[5] * e.p2;
      T *= one_a;
      const float sum = quad_sum9(c, lane);
      if (writes) my_pool[slot * kG] = sum;
    };
    // rounds over the staged records: as many of the next ones as the pool has room for
    for (int k0 = 0, used = 0; k0 < nb;) {
      constexpr uint32_t kNull = (uint32_t)(BATCH - 1) | ((uint32_t)Lds::kPool << KB);
      ListQuad* lp = reinterpret_cast<ListQuad*>(&lds.list[wid][0][0]);
      for (int k = lane; k < 4 * Lds::kStride * 2 / 16; k += 64) lp[k] = (ListQuad)(kNull * 0x10001u);
      int k1 = 0;  // end of the round's records
      int c0 = 0, c1 = 0, c2 = 0, c3 = 0;
#pragma unroll
      for (int h = 0; h < BATCH / 64; ++h) {
        const int k = h * 64 + lane;
        const int first = hit_end[h] - (int)__popc(hits[h]) - used;
        const bool fits = hit_end[h] - used <= Lds::kPool;
        k1 += (int)__popcll(__ballot(fits));
        const uint32_t mine = (fits & (k >= k0)) ? (hits[h] >> (4 * wid)) & 15u : 0u;
        const int slot = first + (int)__popc(hits[h] & ((1u << (4 * wid)) - 1u));
        auto append = [&](int g, int& c) {
          const bool hit = (mine >> g) & 1u;
          const uint64_t m = __ballot(hit);
          if (hit)
            lds.list[wid][g][c + (int)lanemask_lt_count(m)] =
                (uint16_t)(k | ((slot + (int)__popc(mine & ((1u << g) - 1u))) << KB));
          c += (int)__popcll(m);
        };
        append(0, c0);
        append(1, c1);
        append(2, c2);
        append(3, c3);
      }
      k1 = min(k1, nb);
      const int max_cnt = max(max(c0, c1), max(c2, c3));
      // two entries of the lane's quadrant list per trip, in one LDS read (past the quadrant's count:
      // the null record and its slot)
      if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)lds.odd) == 0, 1)) {
        for (int t = 0; t < max_cnt; t += 2) {
          const uint32_t pk = *reinterpret_cast<const ListWord*>(&my_list[t]);
          const uint32_t ka = pk & (BATCH - 1), kb = (pk >> 16) & (BATCH - 1);
          const uint32_t sa = (pk & 0xFFFFu) >> KB, sb = pk >> (16 + KB);
          const float a0 = s_du[ka], b0 = s_du[kb];
          const float4 af = s_f[ka], a1 = s_w1[ka], a2 = s_w2[ka];
          const float4 bf = s_f[kb], b1 = s_w1[kb], b2 = s_w2[kb];
          step(std::false_type{}, ka, sa, a0, af, a1, a2);
          step(std::false_type{}, kb, sb, b0, bf, b1, b2);
        }
      } else {  // one at a time (so that the loop needs no register that the other one does not)
        for (int t = 0; t < max_cnt; ++t) {
          const uint32_t e = my_list[t], k = e & (BATCH - 1);
          step(std::true_type{}, k, e >> KB, s_du[k], s_f[k], s_w1[k], s_w2[k]);
        }
      }
      __syncthreads();
      const int end_used = lds.end[k1 - 1];
      for (uint32_t t = threadIdx.x; t < (uint32_t)((k1 - k0) * kG); t += NT) {
        const uint32_t kk = t / kG, q = t - kk * kG, k = (uint32_t)k0 + kk;
        const int n = (int)__popc(lds.hits((int)k));
        const float* p = s_pool + (uint32_t)((int)lds.end[k] - n - used) * kG + q;
        float v = 0.0f;
        for (int h = 0; h < n; ++h, p += kG) v += *p;
        if constexpr (DET) {
          const float4 f = s_f[k];
          const int64_t slot = det_slot<TW, TH>(det, s_rec[k], (int)f.x, (int)(f.x + f.z), (int)f.y, txi, tyi);
          if (slot < det.slots) det.partial[slot * kG + q] = flush_value(q, v, s_w1[k], s_w2[k]);
        } else {
          v = flush_value(q, v, s_w1[k], s_w2[k]);
          if (v != 0.0f) unsafeAtomicAdd(&grad2d[(int64_t)s_rec[k] * kG + q], v);
        }
      }
      used = end_used;
      k0 = k1;
      __syncthreads();
    }
  }
  if constexpr (DET) {
    // entries behind every pixel's last one were not walked: their slots get zeros
    const uint32_t len = ranges[2 * tile_g + 1] - start;
    for (uint32_t k = (uint32_t)tile_last + threadIdx.x; k < len; k += NT) {
      const uint32_t rid = pair_records[start + k];
      const uint4 w0 = *reinterpret_cast<const uint4*>(&records[rid]);
      const int64_t slot = det_slot<TW, TH>(det, rid, (int)(w0.z & 0xFFFFu),
                                            (int)((w0.z & 0xFFFFu) + (w0.z >> 16)), (int)(w0.w & 0xFFFFu), txi, tyi);
      if (slot < det.slots)
#pragma unroll
        for (int q = 0; q < kG; ++q) det.partial[slot * kG + q] = 0.0f;
    }
  }
}

template <int TW, int TH, int BATCH, bool DET>
__global__ void __launch_bounds__(TW* TH) __attribute__((amdgpu_waves_per_eu(TW * TH >= 128 ? 6 : 1)))
raster_bwd_kernel(TileArgs ta, uint32_t* queue,
                                                            const float* __restrict__ rgb,
                                                            const float* __restrict__ T_final,
                                                            const int32_t* __restrict__ n_last,
                                                            const float* __restrict__ d_rgb,
                                                            float* __restrict__ grad2d, DetArgs det) {
  __shared__ BwdLds<TW, TH, BATCH> lds;
  static_assert(TW * TH != 256 || 6 * sizeof(lds) <= 160 * 1024, "six work-groups per CU");
  for_each_tile(ta, queue, 1, [&](int tile_g) {
    raster_bwd_tile<TW, TH, BATCH, DET>(ta, lds, tile_g, rgb, T_final, n_last, d_rgb, grad2d, det);
  });
}

// ---------------------------------------------------------------------------
// deterministic mode: slots per record, then per-record sums in tile order
// ---------------------------------------------------------------------------
__device__ __forceinline__ int64_t det_pairs(const int64_t* counts, int64_t slots) {
  const int64_t m = counts[GS_COUNT_PAIRS];
  return m < slots ? m : slots;
}

// cnt[r] = 0 for every record, and the slot cursor
__global__ void det_clear_kernel(uint32_t* __restrict__ cnt, uint32_t* __restrict__ cursor, const int64_t* counts,
                                 int64_t cap) {
  int64_t n = counts[GS_COUNT_RECORDS];
  if (n > cap) n = cap;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t0 == 0) *cursor = 0u;
  for (int64_t k = t0; k < n; k += stride) cnt[k] = 0u;
}

// cnt[r] = number of (tile, record) pairs of record r (integer adds: exact in any order)
__global__ void det_count_kernel(const uint32_t* __restrict__ pair_records, const int64_t* counts, int64_t slots,
                                 uint32_t* __restrict__ cnt) {
  const int64_t m = det_pairs(counts, slots);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < m; p += stride)
    atomicAdd(&cnt[pair_records[p]], 1u);
}

// base[r]: a contiguous run of cnt[r] slots per record.  Where a run lies does
// not change any sum, so work-groups take their ranges with one atomic each.
__global__ void __launch_bounds__(256) det_base_kernel(const uint32_t* __restrict__ cnt, const int64_t* counts,
                                                       int64_t cap, uint32_t* __restrict__ cursor,
                                                       uint32_t* __restrict__ base) {
  __shared__ uint32_t s_wave[4];
  __shared__ uint32_t s_start;
  int64_t n = counts[GS_COUNT_RECORDS];
  if (n > cap) n = cap;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  for (int64_t r0 = (int64_t)blockIdx.x * 256; r0 < n; r0 += (int64_t)gridDim.x * 256) {
    const int64_t r = r0 + threadIdx.x;
    const uint32_t c = r < n ? cnt[r] : 0u;
    uint32_t inc = c;
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t y = __shfl_up(inc, off, 64);
      if (lane >= off) inc += y;
    }
    if (lane == 63) s_wave[wid] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
    for (int w = 0; w < 4; ++w) {
      before += w < wid ? s_wave[w] : 0u;
      total += s_wave[w];
    }
    if (threadIdx.x == 0) s_start = total ? atomicAdd(cursor, total) : 0u;
    __syncthreads();
    if (r < n) base[r] = s_start + before + inc - c;
    __syncthreads();
  }
}

// grad2d[r] = sum of record r's slots, in ascending tile order
__global__ void det_reduce_kernel(const float* __restrict__ partial, const uint32_t* __restrict__ cnt,
                                  const uint32_t* __restrict__ base, const int64_t* counts, int64_t cap,
                                  int64_t slots, float* __restrict__ grad2d) {
  int64_t n = counts[GS_COUNT_RECORDS];
  if (n > cap) n = cap;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += stride) {
    const uint32_t c = cnt[r];
    if (c == 0) continue;
    const int64_t b = base[r];
    if (b + c > slots) continue;  // the workspace holds fewer slots than pairs
    float acc[kG];
#pragma unroll
    for (int q = 0; q < kG; ++q) acc[q] = 0.0f;
    for (uint32_t k = 0; k < c; ++k)
#pragma unroll
      for (int q = 0; q < kG; ++q) acc[q] += partial[(b + k) * kG + q];
#pragma unroll
    for (int q = 0; q < kG; ++q) grad2d[r * kG + q] = acc[q];
  }
}

// ---------------------------------------------------------------------------
// preprocess adjoint: per record, chain the 2D partials back to the parameters
// ---------------------------------------------------------------------------
struct BwdArgs {
  LevelPtrs lv[kMaxLevels];
  gs_gaussian_grads gr[kMaxLevels];
  const int64_t* lvl_off;
  const int64_t* lvl_cnt;
  const int8_t* level;
  const int64_t* offsets;
  const uint32_t* gather;  // point-wise selection: record -> index within its level (packed: see below)
  const gs_camera* cams;
  int64_t capacity;
  int32_t B, L, V, W, H, sh_degree;
  int32_t segs;    // segments per view: B (block-wise), L (point-wise) or 1 (packed)
  int32_t packed;  // gather entries are level << GS_PACKED_INDEX_BITS | index (refined selection)
};

// The projection adjoint is bound by its reads and writes of whole parameter planes (1M Gaussians,
// 117K visible in one view: 640 MB of lines touched in 217 us, 46 us of it VALU time).  So:
//  * a Gaussian's parameters are loaded together, ahead of all arithmetic, and ahead of the first store
//    or atomic (vector memory operations are waited for in order: a load behind a store waits for it);
//  * the compositing kernel drops the colour partials of clamped channels, so no record is read here
//    (16 views x 2M: 1 GB of record lines less);
//  * in the Gaussian-major kernel the parameters are read once for all views, and the next view's 2D
//    gradient is in flight during a view's adjoint;
//  * camera and level pointers are scalar (they are one for nearly every wave).
// 1M: 217 -> 156 us; 16 shared views x 2M (12.6M visible): 1041 -> 586 us (2.5 GB, 4.3 TB/s; with vector
// cameras and levels 172 and 637); four views of 262K visible with atomics: 290 -> 270 us, bound by the
// 62M memory-side atomic adds.  Packing the visible records of 1024 into full waves first measured no gain.
//
// Parameters of one Gaussian, loaded together (the loads are all in flight at once).
struct GaussianIn {
  float m[3], q[4], s[3], f[48];  // f: SH coefficient planes of the bands evaluated (f[0..2] unused)
  int deg;                        // SH bands evaluated
  template <bool HALF>
  __device__ __forceinline__ void load(const LevelPtrs& L, int sh_degree, int64_t gi) {
    deg = sh_degree < L.sh_deg ? sh_degree : L.sh_deg;
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] = L.means[k * L.n + gi];
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = attr<HALF>(L.quats, k * L.n + gi);
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] = attr<HALF>(L.scales, k * L.n + gi);
    const int terms = 3 * (deg + 1) * (deg + 1);
#pragma unroll
    for (int i = 3; i < 48; ++i) f[i] = i < terms ? attr<HALF>(L.sh, (int64_t)i * L.n + gi) : 0.0f;
  }
};

// Gradient of one record's parameters.  The SH part (dL/df_{k,c} = Y_k g_c) is left as its factors:
// a destination forms the 48 products as it stores or sums them.
struct RecordGrad {
  float dir[3], g[3];  // view direction, colour gradient
  int deg;             // SH bands evaluated
  float m[3], s[3], q[4], o;
};

// SH basis up to degree `deg` at a unit direction: f(k, Y_k, dY_k/dx, dY_k/dy, dY_k/dz) per term
// (what the callback does not use is never computed).
template <class F>
__device__ __forceinline__ void sh_terms(float x, float y, float z, int deg, F f) {
  const float k1 = (float)kSH1, k2a = (float)kSH2a, k2b = (float)kSH2b, k2c = (float)kSH2c;
  const float k3a = (float)kSH3a, k3b = (float)kSH3b, k3c = (float)kSH3c, k3d = (float)kSH3d, k3e = (float)kSH3e;
  f(0, (float)kSH00, 0.f, 0.f, 0.f);
  if (deg < 1) return;
  f(1, -k1 * y, 0.f, -k1, 0.f);
  f(2, k1 * z, 0.f, 0.f, k1);
  f(3, -k1 * x, -k1, 0.f, 0.f);
  if (deg < 2) return;
  const float xx = x * x, yy = y * y, zz = z * z;
  f(4, k2a * x * y, k2a * y, k2a * x, 0.f);
  f(5, -k2a * y * z, 0.f, -k2a * z, -k2a * y);
  f(6, k2b * (2.f * zz - xx - yy), -2.f * k2b * x, -2.f * k2b * y, 4.f * k2b * z);
  f(7, -k2a * x * z, -k2a * z, 0.f, -k2a * x);
  f(8, k2c * (xx - yy), 2.f * k2c * x, -2.f * k2c * y, 0.f);
  if (deg < 3) return;
  f(9, -k3a * y * (3.f * xx - yy), -6.f * k3a * x * y, -3.f * k3a * (xx - yy), 0.f);
  f(10, k3b * x * y * z, k3b * y * z, k3b * x * z, k3b * x * y);
  f(11, -k3c * y * (4.f * zz - xx - yy), 2.f * k3c * x * y, -k3c * (4.f * zz - xx - 3.f * yy), -8.f * k3c * y * z);
  f(12, k3d * z * (2.f * zz - 3.f * xx - 3.f * yy), -6.f * k3d * x * z, -6.f * k3d * y * z,
    k3d * (6.f * zz - 3.f * xx - 3.f * yy));
  f(13, -k3c * x * (4.f * zz - xx - yy), -k3c * (4.f * zz - 3.f * xx - yy), 2.f * k3c * x * y, -8.f * k3c * x * z);
  f(14, k3e * z * (xx - yy), 2.f * k3e * x * z, -2.f * k3e * y * z, k3e * (xx - yy));
  f(15, -k3a * x * (xx - 3.f * yy), -3.f * k3a * (xx - yy), 6.f * k3a * x * y, 0.f);
}

// Destinations.  All of a record's loads come before its first store or atomic
// (vector memory operations are waited for in order, so a load behind a store
// waits for it): the SH coefficients were read for the direction gradient already
// and the products need only the direction.
//
// add_atomic: no-return FP32 atomics (records of one Gaussian may run
// concurrently when views share it).
__device__ __forceinline__ void add_atomic(const gs_gaussian_grads& G, int64_t n, int64_t gi, const RecordGrad& r) {
  sh_terms(r.dir[0], r.dir[1], r.dir[2], r.deg, [&](int k, float Y, float, float, float) {
#pragma unroll
    for (int c = 0; c < 3; ++c) unsafeAtomicAdd(&G.sh[(int64_t)(3 * k + c) * n + gi], Y * r.g[c]);
  });
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    unsafeAtomicAdd(&G.means[k * n + gi], r.m[k]);
    unsafeAtomicAdd(&G.scales[k * n + gi], r.s[k]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) unsafeAtomicAdd(&G.quats[k * n + gi], r.q[k]);
  unsafeAtomicAdd(&G.opac[gi], r.o);
}

// add_plain: the only record of its Gaussian in the launch (one view).
__device__ __forceinline__ void add_plain(const gs_gaussian_grads& G, int64_t n, int64_t gi, const RecordGrad& r) {
  float cm[3], cs[3], cq[4], csh[48];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    cm[k] = G.means[k * n + gi];
    cs[k] = G.scales[k * n + gi];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) cq[k] = G.quats[k * n + gi];
  const float co = G.opac[gi];
  const int terms = 3 * (r.deg + 1) * (r.deg + 1);
#pragma unroll
  for (int i = 0; i < 48; ++i) csh[i] = i < terms ? G.sh[(int64_t)i * n + gi] : 0.0f;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    G.means[k * n + gi] = cm[k] + r.m[k];
    G.scales[k * n + gi] = cs[k] + r.s[k];
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) G.quats[k * n + gi] = cq[k] + r.q[k];
  G.opac[gi] = co + r.o;
  sh_terms(r.dir[0], r.dir[1], r.dir[2], r.deg, [&](int k, float Y, float, float, float) {
#pragma unroll
    for (int c = 0; c < 3; ++c) G.sh[(int64_t)(3 * k + c) * n + gi] = csh[3 * k + c] + Y * r.g[c];
  });
}

// RegisterSink sums the gradients of all records of one Gaussian (a thread
// that owns them, views in order) and adds the totals to memory once.
struct RegisterSink {
  float shv[48], m[3], s[3], q[4], o;
  __device__ __forceinline__ RegisterSink() {
#pragma unroll
    for (int i = 0; i < 48; ++i) shv[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 3; ++i) m[i] = s[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = 0.0f;
    o = 0.0f;
  }
  __device__ __forceinline__ void sh(int i, float v) { shv[i] += v; }
  __device__ __forceinline__ void add(const RecordGrad& r) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      m[k] += r.m[k];
      s[k] += r.s[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] += r.q[k];
    o += r.o;
  }
  // planes: coefficient planes stored per colour channel ((sh_degree + 1)^2).
  // Every current value is loaded before the first store, so the loads are in
  // flight together (in a += chain each load would wait for the previous store).
  __device__ __forceinline__ void flush(const gs_gaussian_grads& G, int64_t n, int64_t gi, int planes) const {
    float cm[3], cs[3], cq[4], csh[48];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      cm[k] = G.means[k * n + gi];
      cs[k] = G.scales[k * n + gi];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) cq[k] = G.quats[k * n + gi];
    const float co = G.opac[gi];
#pragma unroll
    for (int i = 0; i < 48; ++i) csh[i] = i < 3 * planes ? G.sh[(int64_t)i * n + gi] : 0.0f;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      G.means[k * n + gi] = cm[k] + m[k];
      G.scales[k * n + gi] = cs[k] + s[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) G.quats[k * n + gi] = cq[k] + q[k];
    G.opac[gi] = co + o;
#pragma unroll
    for (int i = 0; i < 48; ++i)
      if (i < 3 * planes) G.sh[(int64_t)i * n + gi] = csh[i] + shv[i];
  }
};

// For destinations that form the SH products themselves (from RecordGrad)
struct NoSh {
  __device__ __forceinline__ void sh(int, float) {}
};

// Record g's 2D gradient (colour, opacity, conic and mean partials); false if
// it is all zero (a culled record, or one no pixel's loss depends on).
__device__ __forceinline__ bool load_grad2d(const float* __restrict__ grad2d, int64_t g, float (&p2)[kG]) {
  bool any = false;
#pragma unroll
  for (int q = 0; q < kG; ++q) {
    p2[q] = grad2d[g * kG + q];
    any |= p2[q] != 0.0f;
  }
  return any;
}

// One record's adjoint, for a record whose 2D gradient p2 is not all zero.
template <class Sink>
__device__ __forceinline__ void preprocess_bwd_record_t(const BwdArgs& a, const GaussianIn& in, const gs_camera& cam,
                                                        const float (&p2)[kG], const ViewConst& vc, RecordGrad& out,
                                                        Sink& sink) {
  // A record with a non-zero 2D gradient was visible in the forward pass, so
  // the projection below (same code, same inputs) takes the same decisions.
  // ---- colour first (FP32; clamped channels come with no gradient)
  double dm_col[3];
  {
    const double d0 = (double)in.m[0] - vc.C[0], d1 = (double)in.m[1] - vc.C[1], d2 = (double)in.m[2] - vc.C[2];
    const double rdn = 1.0 / sqrt((d0 * d0 + d1 * d1) + d2 * d2);
    const float dir[3] = {(float)(d0 * rdn), (float)(d1 * rdn), (float)(d2 * rdn)};
    const float g[3] = {p2[0], p2[1], p2[2]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      out.dir[k] = dir[k];
      out.g[k] = g[k];
    }
    out.deg = in.deg;
    float gdir[3] = {0.0f, 0.0f, 0.0f};
    sh_terms(dir[0], dir[1], dir[2], in.deg, [&](int k, float Y, float dx, float dy, float dz) {
      if (k > 0) {  // (the constant term has no derivative)
        const float w = fmaf(g[0], in.f[3 * k], fmaf(g[1], in.f[3 * k + 1], g[2] * in.f[3 * k + 2]));
        gdir[0] = fmaf(w, dx, gdir[0]);
        gdir[1] = fmaf(w, dy, gdir[1]);
        gdir[2] = fmaf(w, dz, gdir[2]);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) sink.sh(3 * k + c, Y * g[c]);
    });
    const float gd = gdir[0] * dir[0] + gdir[1] * dir[1] + gdir[2] * dir[2];
    for (int k = 0; k < 3; ++k) dm_col[k] = (double)(gdir[k] - dir[k] * gd) * rdn;
  }
  // ---- geometry adjoint (FP32); the guard-band clamp is decided in FP64 exactly as in the forward pass
  const double* R64 = cam.R;
  const double m0 = in.m[0], m1 = in.m[1], m2 = in.m[2];
  const double tx64 = ((R64[0] * m0 + R64[1] * m1) + R64[2] * m2) + cam.t[0];
  const double ty64 = ((R64[3] * m0 + R64[4] * m1) + R64[5] * m2) + cam.t[1];
  const double tz64 = ((R64[6] * m0 + R64[7] * m1) + R64[8] * m2) + cam.t[2];
  const double rz64 = 1.0 / tz64;
  const double ux64 = tx64 * rz64, uy64 = ty64 * rz64;
  const double uxc64 = dmin_(vc.limx, dmax_(-vc.limx, ux64)), uyc64 = dmin_(vc.limy, dmax_(-vc.limy, uy64));
  const bool clamp_x = uxc64 != ux64, clamp_y = uyc64 != uy64;
  const float tx = (float)tx64, ty = (float)ty64, rz = (float)rz64;
  const float uxc = (float)uxc64, uyc = (float)uyc64;
  const float fx = (float)cam.fx, fy = (float)cam.fy;
  float Rc[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) Rc[k] = (float)R64[k];
  // rotation of the normalised quaternion, scales
  const float qa = in.q[0], qb = in.q[1], qc = in.q[2], qd_ = in.q[3];
  const float qinv = 1.0f / sqrtf(qa * qa + qb * qb + qc * qc + qd_ * qd_);
  const float w = qa * qinv, x = qb * qinv, y = qc * qinv, z = qd_ * qinv;
  float Rq[3][3];
  Rq[0][0] = 1.f - 2.f * (y * y + z * z);
  Rq[0][1] = 2.f * (x * y - w * z);
  Rq[0][2] = 2.f * (x * z + w * y);
  Rq[1][0] = 2.f * (x * y + w * z);
  Rq[1][1] = 1.f - 2.f * (x * x + z * z);
  Rq[1][2] = 2.f * (y * z - w * x);
  Rq[2][0] = 2.f * (x * z - w * y);
  Rq[2][1] = 2.f * (y * z + w * x);
  Rq[2][2] = 1.f - 2.f * (x * x + y * y);
  const float sc[3] = {in.s[0], in.s[1], in.s[2]};
  float WL[3][3];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      WL[i][j] = (Rc[3 * i] * Rq[0][j] + Rc[3 * i + 1] * Rq[1][j] + Rc[3 * i + 2] * Rq[2][j]) * sc[j];
  const float J00 = fx * rz, J02 = -(fx * uxc) * rz, J11 = fy * rz, J12 = -(fy * uyc) * rz;
  float M[2][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    M[0][j] = J00 * WL[0][j] + J02 * WL[2][j];
    M[1][j] = J11 * WL[1][j] + J12 * WL[2][j];
  }
  const float n0 = M[0][0] * M[0][0] + M[0][1] * M[0][1] + M[0][2] * M[0][2];
  const float n1 = M[1][0] * M[1][0] + M[1][1] * M[1][1] + M[1][2] * M[1][2];
  const float sb = M[0][0] * M[1][0] + M[0][1] * M[1][1] + M[0][2] * M[1][2];
  const float sc2 = n1 + 0.3f;
  const float cr0 = M[0][1] * M[1][2] - M[0][2] * M[1][1];
  const float cr1 = M[0][2] * M[1][0] - M[0][0] * M[1][2];
  const float cr2 = M[0][0] * M[1][1] - M[0][1] * M[1][0];
  const float det = cr0 * cr0 + cr1 * cr1 + cr2 * cr2 + 0.3f * (n0 + n1) + 0.09f;
  // ---- 2D mean and conic partials ----
  // F = kS F0 = kS [[ca, cb], [0, cc]]
  const float kS = (float)kConicScale;
  const float ca = sqrtf(sc2 / det);
  const float cb = -sb / sqrtf(sc2 * det);
  const float cc = 1.0f / sqrtf(sc2);
  const float gu = -2.0f * kS * (ca * p2[4]);
  const float gv = -2.0f * kS * (cb * p2[4] + cc * p2[5]);
  // conic K = Sigma2D^-1 = F0^T F0: dL/dSigma = -K (kS^2 sum w d d^T) K = -F0^T P F0
  // with P the second moments of p = F d
  const float P11 = p2[6], P12 = p2[7], P22 = p2[8];
  const float h2 = fmaf(cb, P11, cc * P12);
  const float h3 = fmaf(cb, P12, cc * P22);
  const float S00 = -ca * ca * P11;
  const float S01 = -ca * h2;
  const float S11 = -fmaf(cb, h2, cc * h3);
  // Sigma2D = M M^T + 0.3 I -> dL/dM = 2 Gs M; M = J WL; WL = R_cam Rq diag(s), one column at a time
  float dJ00 = 0.f, dJ02 = 0.f, dJ11 = 0.f, dJ12 = 0.f;
  float ds[3], dRq[3][3];
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    const float dM0 = 2.0f * (S00 * M[0][j] + S01 * M[1][j]);
    const float dM1 = 2.0f * (S01 * M[0][j] + S11 * M[1][j]);
    dJ00 += dM0 * WL[0][j];
    dJ02 += dM0 * WL[2][j];
    dJ11 += dM1 * WL[1][j];
    dJ12 += dM1 * WL[2][j];
    const float dW0 = J00 * dM0, dW1 = J11 * dM1, dW2 = J02 * dM0 + J12 * dM1;
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const float dLm = Rc[i] * dW0 + Rc[3 + i] * dW1 + Rc[6 + i] * dW2;  // (R_cam^T dWL)[i][j]
      acc += Rq[i][j] * dLm;
      dRq[i][j] = sc[j] * dLm;
    }
    ds[j] = acc;
  }
  float dq[4];
  dq[0] = 2.f * (-z * dRq[0][1] + y * dRq[0][2] + z * dRq[1][0] - x * dRq[1][2] - y * dRq[2][0] + x * dRq[2][1]);
  dq[1] = 2.f * (y * dRq[0][1] + z * dRq[0][2] + y * dRq[1][0] - w * dRq[1][2] + z * dRq[2][0] + w * dRq[2][1]) -
          4.f * x * (dRq[1][1] + dRq[2][2]);
  dq[2] = 2.f * (x * dRq[0][1] + w * dRq[0][2] + x * dRq[1][0] + z * dRq[1][2] - w * dRq[2][0] + z * dRq[2][1]) -
          4.f * y * (dRq[0][0] + dRq[2][2]);
  dq[3] = 2.f * (-w * dRq[0][1] + x * dRq[0][2] + w * dRq[1][0] + y * dRq[1][2] + x * dRq[2][0] + y * dRq[2][1]) -
          4.f * z * (dRq[0][0] + dRq[1][1]);
  const float qdot = w * dq[0] + x * dq[1] + y * dq[2] + z * dq[3];
  const float qn[4] = {w, x, y, z};
#pragma unroll
  for (int k = 0; k < 4; ++k) out.q[k] = (dq[k] - qn[k] * qdot) * qinv;
  // J(t) and (u, v)(t)
  const float rz2 = rz * rz;
  float dt0 = gu * fx * rz, dt1 = gv * fy * rz;
  float dt2 = -gu * fx * tx * rz2 - gv * fy * ty * rz2 - dJ00 * fx * rz2 - dJ11 * fy * rz2;
  if (!clamp_x) {
    dt0 += -dJ02 * fx * rz2;
    dt2 += dJ02 * 2.0f * fx * tx * rz2 * rz;
  } else {
    dt2 += dJ02 * fx * uxc * rz2;
  }
  if (!clamp_y) {
    dt1 += -dJ12 * fy * rz2;
    dt2 += dJ12 * 2.0f * fy * ty * rz2 * rz;
  } else {
    dt2 += dJ12 * fy * uyc * rz2;
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    out.m[k] = Rc[k] * dt0 + Rc[3 + k] * dt1 + Rc[6 + k] * dt2 + (float)dm_col[k];
    out.s[k] = ds[k];
  }
  out.o = p2[3];
}

// All records of Gaussian gi (index i in every view's selection), views in
// order, summed in registers and added to memory once.  The Gaussian's
// parameters are read once; the next view's 2D gradient is in flight while a
// view's adjoint is computed.
template <bool HALF>
__device__ __forceinline__ void preprocess_bwd_gaussian(const BwdArgs& a, const float* __restrict__ grad2d,
                                                        int64_t n_rec, int64_t n_view, int64_t i, int l, int64_t gi,
                                                        const ViewConst (&s_view)[kLdsViews]) {
  if (i >= n_rec) return;
  float p2[kG];
  bool hit = load_grad2d(grad2d, i, p2);
  GaussianIn in;
  in.load<HALF>(a.lv[l], a.sh_degree, gi);
  RegisterSink acc;
  bool any = false;
  int64_t g = i;
  for (int v = 0; v < a.V; ++v, g += n_view) {
    if (g >= n_rec) break;
    float next[kG] = {};
    const bool more = v + 1 < a.V && g + n_view < n_rec;
    bool next_hit = false;
    if (more) next_hit = load_grad2d(grad2d, g + n_view, next);
    if (hit) {
      RecordGrad r;
      preprocess_bwd_record_t(a, in, uniform_camera(a.cams, v), p2, view_const(a.cams, a.V, a.W, a.H, s_view, v), r, acc);
      acc.add(r);
      any = true;
    }
    hit = next_hit;
#pragma unroll
    for (int q = 0; q < kG; ++q) p2[q] = next[q];
  }
  if (any) acc.flush(a.gr[l], a.lv[l].n, gi, (a.lv[l].sh_deg + 1) * (a.lv[l].sh_deg + 1));
}

// View-major: records in index order, gradients added with no-return atomics
// (SINGLE: one view, each Gaussian has at most one record: register sums
// flushed with all loads ahead of the stores).
template <bool SINGLE>
__global__ void __launch_bounds__(256) preprocess_bwd_kernel(BwdArgs a, const float* __restrict__ grad2d,
                                                             const int64_t* __restrict__ counts) {
  int64_t n_rec = counts[GS_COUNT_RECORDS];
  if (n_rec > a.capacity) n_rec = a.capacity;
  const int nseg = a.V * a.segs;
  // segment offsets staged in LDS when they fit; a record is looked up only
  // once its 2D gradient is known to be non-zero (most selected records were culled)
  __shared__ int64_t s_off[kBwdLdsOffsets];
  __shared__ ViewConst s_view[kLdsViews];
  load_views(a.cams, a.V, a.W, a.H, s_view);
  const bool lds_off = nseg < kBwdLdsOffsets;
  if (lds_off)
    for (int k = threadIdx.x; k <= nseg; k += blockDim.x) s_off[k] = a.offsets[k];
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n_rec; g += stride) {
    float p2[kG];
    const uint32_t entry = a.gather ? a.gather[g] : 0u;  // (in flight with the gradient)
    if (!load_grad2d(grad2d, g, p2)) continue;
    const int p = lds_off ? find_segment(s_off, nseg, g) : find_segment(a.offsets, nseg, g);
    const int v = p / a.segs, b = p - v * a.segs;
    int l;
    int64_t gi;
    if (a.packed) {  // refined selection: the entry names the level and the index
      l = (int)(entry >> GS_PACKED_INDEX_BITS);
      gi = (int64_t)(entry & ((1u << GS_PACKED_INDEX_BITS) - 1u));
      if (l >= a.L || gi >= a.lv[l].n) continue;  // not a stored Gaussian (the forward culled it)
    } else {
      l = a.gather ? b : a.level[p];
      const int64_t seg0 = lds_off ? s_off[p] : a.offsets[p];
      gi = a.gather ? (int64_t)entry : a.lvl_off[(int64_t)b * a.L + l] + (g - seg0);
    }
    for_each_key(v * kMaxLevels + l, [&](int key) {
      const int uv = key / kMaxLevels, ul = key % kMaxLevels;
      const LevelPtrs& L = a.lv[ul];
      GaussianIn in;
      if (L.half) in.load<true>(L, a.sh_degree, gi);
      else in.load<false>(L, a.sh_degree, gi);
      RecordGrad r;
      NoSh none;
      preprocess_bwd_record_t(a, in, uniform_camera(a.cams, uv), p2, view_const(a.cams, a.V, a.W, a.H, s_view, uv), r,
                              none);
      if constexpr (SINGLE) add_plain(a.gr[ul], L.n, gi, r);
      else add_atomic(a.gr[ul], L.n, gi, r);
    });
  }
}

// Gaussian-major (every view selected the same records): one thread owns a
// Gaussian's records in all views and sums its gradient in registers.
__global__ void __launch_bounds__(256) preprocess_bwd_shared_kernel(BwdArgs a, const float* __restrict__ grad2d,
                                                                    const int64_t* __restrict__ counts) {
  if (counts[GS_COUNT_FLAGS] & GS_FLAG_SELECTION) return;  // the forward projected nothing
  int64_t n_rec = counts[GS_COUNT_RECORDS];
  if (n_rec > a.capacity) n_rec = a.capacity;
  __shared__ ViewConst s_view[kLdsViews];
  load_views(a.cams, a.V, a.W, a.H, s_view);
  __syncthreads();
  const int64_t n_view = a.offsets[a.segs];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_view; i += stride) {
    const int b = find_segment(a.offsets, a.segs, i);
    const int l = a.gather ? b : a.level[b];
    const int64_t gi = a.gather ? (int64_t)a.gather[i] : a.lvl_off[(int64_t)b * a.L + l] + (i - a.offsets[b]);
    for_each_key(l, [&](int u) {
      if (a.lv[u].half) preprocess_bwd_gaussian<true>(a, grad2d, n_rec, n_view, i, u, gi, s_view);
      else preprocess_bwd_gaussian<false>(a, grad2d, n_rec, n_view, i, u, gi, s_view);
    });
  }
}

// Deterministic mode with several views that selected different blocks or
// levels (block-wise): one thread per stored Gaussian of every level sums its
// records over the views in view order (record of view v: the view chose the
// Gaussian's block at the Gaussian's level) and adds the total once.
__global__ void __launch_bounds__(256) preprocess_bwd_det_kernel(BwdArgs a, const float* __restrict__ grad2d,
                                                                 const int64_t* __restrict__ counts,
                                                                 int64_t n_stored) {
  int64_t n_rec = counts[GS_COUNT_RECORDS];
  if (n_rec > a.capacity) n_rec = a.capacity;
  __shared__ ViewConst s_view[kLdsViews];
  load_views(a.cams, a.V, a.W, a.H, s_view);
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_stored; t += stride) {
    int l = 0;
    int64_t gi = t;
    while (l < a.L - 1 && gi >= a.lv[l].n) gi -= a.lv[l++].n;
    // block of gi in level l: blocks are stored in block order, so the last block
    // whose first index is <= gi (then checked against its count)
    int lo = 0, hi = a.B - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (a.lvl_off[(int64_t)mid * a.L + l] <= gi) lo = mid;
      else hi = mid - 1;
    }
    const int b = lo;
    const int64_t first = a.lvl_off[(int64_t)b * a.L + l];
    if (gi < first || gi >= first + a.lvl_cnt[(int64_t)b * a.L + l]) continue;
    RegisterSink acc;
    bool any = false;
    for (int v = 0; v < a.V; ++v) {
      const int64_t p = (int64_t)v * a.B + b;
      if (a.level[p] != l) continue;
      const int64_t g = a.offsets[p] + (gi - first);
      if (g >= n_rec) continue;
      float p2[kG];
      if (!load_grad2d(grad2d, g, p2)) continue;
      GaussianIn in;
      if (a.lv[l].half) in.load<true>(a.lv[l], a.sh_degree, gi);
      else in.load<false>(a.lv[l], a.sh_degree, gi);
      RecordGrad r;
      preprocess_bwd_record_t(a, in, a.cams[v], p2, view_const(a.cams, a.V, a.W, a.H, s_view, v), r, acc);
      acc.add(r);
      any = true;
    }
    if (any) acc.flush(a.gr[l], a.lv[l].n, gi, (a.lv[l].sh_deg + 1) * (a.lv[l].sh_deg + 1));
  }
}

__global__ void clear_floats_kernel(float* __restrict__ p, const int64_t* counts, int64_t cap, int per_record) {
  int64_t n = counts[GS_COUNT_RECORDS];
  if (n > cap) n = cap;
  const int64_t words = n * per_record;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < words; k += stride) p[k] = 0.0f;
}

template <int TW, int TH>
void launch_bwd(int batch, bool det, const TileArgs& ta, uint32_t* queue, hipStream_t s, const float* rgb,
                const float* T, const int32_t* nl, const float* drgb, float* g2d, const DetArgs& d) {
  constexpr int NT = TW * TH;
  const dim3 grid = tile_grid(ta.n_tiles, queue != nullptr);
  // at most 128 staged records: a larger batch would only wait for room in the pool
  if (batch == 64 && det)
    hipLaunchKernelGGL((raster_bwd_kernel<TW, TH, 64, true>), grid, dim3(NT), 0, s, ta, queue, rgb, T, nl, drgb, g2d,
                       d);
  else if (batch == 64)
    hipLaunchKernelGGL((raster_bwd_kernel<TW, TH, 64, false>), grid, dim3(NT), 0, s, ta, queue, rgb, T, nl, drgb,
                       g2d, d);
  else if (det)
    hipLaunchKernelGGL((raster_bwd_kernel<TW, TH, 128, true>), grid, dim3(NT), 0, s, ta, queue, rgb, T, nl, drgb,
                       g2d, d);
  else
    hipLaunchKernelGGL((raster_bwd_kernel<TW, TH, 128, false>), grid, dim3(NT), 0, s, ta, queue, rgb, T, nl, drgb,
                       g2d, d);
}

// workspace: grad2d [rc][kG]; deterministic mode adds cnt [rc], base [rc], a
// cursor and partial [slots][kG] with one slot per pair of pair capacity
struct BwdWs {
  float* grad2d;
  uint32_t* cnt;
  uint32_t* base;
  uint32_t* cursor;
  float* partial;
  size_t fixed_bytes;  // everything but the slots
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

BwdWs bwd_ws_layout(char* p, int64_t rc, bool det) {
  BwdWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* q = p ? p + off : nullptr;
    off = align256(off + bytes);
    return q;
  };
  w.grad2d = (float*)take((size_t)rc * kG * sizeof(float));
  if (det) {
    w.cnt = (uint32_t*)take((size_t)rc * 4);
    w.base = (uint32_t*)take((size_t)rc * 4);
    w.cursor = (uint32_t*)take(4);
    w.partial = (float*)(p ? p + off : nullptr);
  }
  w.fixed_bytes = off;
  return w;
}

}  // namespace

size_t rasterize_bwd_ws_bytes(int64_t rc, int64_t pc, bool det) {
  const size_t fixed = bwd_ws_layout(nullptr, rc, det).fixed_bytes;
  return det ? fixed + (size_t)pc * kG * sizeof(float) : fixed + 256;
}

}  // namespace gs

extern "C" gs_status gs_rasterize_bwd(const void* records, const uint32_t* pair_records, const uint32_t* tile_ranges,
                                      uint32_t* tile_queue, int32_t n_views, int32_t width, int32_t height,
                                      const float* bg,
                                      const gs_tuning* tuning, const float* rgb, const float* T_final,
                                      const int32_t* n_last, const float* d_rgb, const gs_gaussians* levels,
                                      const gs_blocks* blocks, const int8_t* level, const int64_t* offsets,
                                      const uint32_t* gather, const gs_camera* cams, int32_t sh_degree,
                                      int64_t record_capacity,
                                      const int64_t* counts, const gs_gaussian_grads* grads, void* ws,
                                      size_t ws_bytes, void* stream) {
  using namespace gs;
  (void)bg;  // the background enters through the saved forward colour
  if (!records || !pair_records || !tile_ranges || !tuning || !rgb || !T_final || !n_last || !d_rgb || !levels ||
      !blocks || (!level && !gather) || !offsets || !cams || !counts || !grads || !ws)
    return GS_ERR_INVALID_ARG;
  if (n_views <= 0 || width <= 0 || height <= 0 || width > 65535 || height > 65535) return GS_ERR_INVALID_ARG;
  if (sh_degree < 0 || sh_degree > 3 || record_capacity <= 0) return GS_ERR_INVALID_ARG;
  if (blocks->n_levels <= 0 || blocks->n_levels > kMaxLevels) return GS_ERR_INVALID_ARG;
  if (!gather && (blocks->n_blocks <= 0 || !blocks->lvl_off)) return GS_ERR_INVALID_ARG;
  const int tw = tuning->tile_w, th = tuning->tile_h;
  if (!tile_shape_supported(tw, th) || !batch_supported(tuning->batch)) return GS_ERR_UNSUPPORTED;
  const bool packed = (tuning->flags & GS_TUNE_PACKED_SELECTION) != 0;
  if (packed && !gather) return GS_ERR_INVALID_ARG;
  const bool det = (tuning->flags & GS_TUNE_DETERMINISTIC) != 0;
  const bool shared = (tuning->flags & GS_TUNE_SHARED_SELECTION) && n_views > 1;
  // decided before any launch: the Gaussian-major adjoint takes block-wise selections only, and the
  // deterministic adjoint of several different selections needs the block-wise level table
  if (shared && gather) return GS_ERR_UNSUPPORTED;
  if (det && gather && n_views > 1 && !shared) return GS_ERR_UNSUPPORTED;
  if (det && !shared && n_views > 1 && !blocks->lvl_cnt) return GS_ERR_INVALID_ARG;
  if (ws_bytes < rasterize_bwd_ws_bytes(record_capacity, 0, det)) return GS_ERR_WORKSPACE;
  const BwdWs w = bwd_ws_layout((char*)ws, record_capacity, det);
  float* grad2d = w.grad2d;
  DetArgs d{};
  if (det) {
    d.partial = w.partial;
    d.base = w.base;
    d.slots = (int64_t)((ws_bytes - w.fixed_bytes) / (kG * sizeof(float)));
  }
  const int tx = tiles_x(width, tw), ty = tiles_y(height, th);
  const int64_t tpv = (int64_t)tx * ty;
  const int64_t nblocks = tpv * n_views;
  if (nblocks >= ((int64_t)1 << 31)) return GS_ERR_INVALID_ARG;
  hipStream_t s = (hipStream_t)stream;
  int64_t cg = (record_capacity * kG + 255) / 256;
  hipLaunchKernelGGL(clear_floats_kernel, dim3((unsigned)(cg < 4096 ? (cg < 1 ? 1 : cg) : 4096)), dim3(256), 0, s,
                     grad2d, counts, record_capacity, kG);
  GS_LAUNCH_CHECK();
  const unsigned rg = (unsigned)(cg < 4096 ? (cg < 1 ? 1 : cg) : 4096);
  if (det) {
    // slots: count each record's pairs, then give each record a run of that many
    hipLaunchKernelGGL(det_clear_kernel, dim3(rg), dim3(256), 0, s, w.cnt, w.cursor, counts, record_capacity);
    hipLaunchKernelGGL(det_count_kernel, dim3(4096), dim3(256), 0, s, pair_records, counts, d.slots, w.cnt);
    hipLaunchKernelGGL(det_base_kernel, dim3(2048), dim3(256), 0, s, w.cnt, counts, record_capacity, w.cursor,
                       w.base);
    GS_LAUNCH_CHECK();
  }
  const Record* rec = (const Record*)records;
  const TileArgs ta{rec, pair_records, tile_ranges, width, height, tx, (int)tpv, nblocks};
  uint32_t* q = ((tuning->flags & GS_TUNE_WORK_QUEUE) && tile_queue) ? tile_queue : nullptr;
  const int b = tuning->batch;
  if (tw == 16 && th == 16) launch_bwd<16, 16>(b, det, ta, q, s, rgb, T_final, n_last, d_rgb, grad2d, d);
  else if (tw == 8 && th == 8) launch_bwd<8, 8>(b, det, ta, q, s, rgb, T_final, n_last, d_rgb, grad2d, d);
  else if (tw == 16 && th == 8) launch_bwd<16, 8>(b, det, ta, q, s, rgb, T_final, n_last, d_rgb, grad2d, d);
  else if (tw == 32 && th == 8) launch_bwd<32, 8>(b, det, ta, q, s, rgb, T_final, n_last, d_rgb, grad2d, d);
  else launch_bwd<32, 16>(b, det, ta, q, s, rgb, T_final, n_last, d_rgb, grad2d, d);
  GS_LAUNCH_CHECK();
  if (det) {
    hipLaunchKernelGGL(det_reduce_kernel, dim3(rg), dim3(256), 0, s, w.partial, w.cnt, w.base, counts,
                       record_capacity, d.slots, grad2d);
    GS_LAUNCH_CHECK();
  }
  BwdArgs a{};
  for (int l = 0; l < blocks->n_levels; ++l) {
    const gs_gaussians& g = levels[l];
    if (g.sh_degree < 0 || g.sh_degree > 3 || (g.attr_half != 0 && g.attr_half != 1)) return GS_ERR_INVALID_ARG;
    a.lv[l] = level_ptrs(g);
    a.gr[l] = grads[l];
    if (g.n > 0 && (!grads[l].means || !grads[l].scales || !grads[l].quats || !grads[l].opac || !grads[l].sh))
      return GS_ERR_INVALID_ARG;
  }
  a.lvl_off = blocks->lvl_off;
  a.lvl_cnt = blocks->lvl_cnt;
  a.level = level;
  a.offsets = offsets;
  a.gather = gather;
  a.segs = packed ? 1 : gather ? blocks->n_levels : blocks->n_blocks;
  a.packed = packed ? 1 : 0;
  a.cams = cams;
  a.capacity = record_capacity;
  a.B = blocks->n_blocks;
  a.L = blocks->n_levels;
  a.V = n_views;
  a.W = width;
  a.H = height;
  a.sh_degree = sh_degree;
  int64_t gb = (record_capacity + 255) / 256;
  const dim3 gbg((unsigned)(gb < 8192 ? (gb < 1 ? 1 : gb) : 8192));
  if ((tuning->flags & GS_TUNE_SHARED_SELECTION) && n_views > 1) {
    if (gather) return GS_ERR_UNSUPPORTED;
    int64_t pv = (record_capacity / n_views + 255) / 256;
    const dim3 gs_grid((unsigned)(pv < 8192 ? (pv < 1 ? 1 : pv) : 8192));
    hipLaunchKernelGGL(preprocess_bwd_shared_kernel, gs_grid, dim3(256), 0, s, a, grad2d, counts);
  } else if (n_views == 1) {
    hipLaunchKernelGGL(preprocess_bwd_kernel<true>, gbg, dim3(256), 0, s, a, grad2d, counts);
  } else if (det) {
    if (!blocks->lvl_cnt) return GS_ERR_INVALID_ARG;
    int64_t n_stored = 0;
    for (int l = 0; l < blocks->n_levels; ++l) n_stored += levels[l].n;
    int64_t sb = (n_stored + 255) / 256;
    const dim3 sg((unsigned)(sb < 8192 ? (sb < 1 ? 1 : sb) : 8192));
    hipLaunchKernelGGL(preprocess_bwd_det_kernel, sg, dim3(256), 0, s, a, grad2d, counts, n_stored);
  } else {
    hipLaunchKernelGGL(preprocess_bwd_kernel<false>, gbg, dim3(256), 0, s, a, grad2d, counts);
  }
  GS_LAUNCH_CHECK();
  return GS_OK;
}
