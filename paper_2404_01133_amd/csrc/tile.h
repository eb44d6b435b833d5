// Pieces shared by the per-tile compositing kernels (forward and adjoint):
// evaluation of a record at a pixel, the lane -> pixel map, per-group record
// lists, the tile arguments and the work distribution over tiles.  Included by
// translation units compiled with -ffp-contract=off: evaluate_f() is the
// operation order both kernels must share.
#pragma once

#include "project.h"

namespace gs {
namespace {

// Value of a projected Gaussian at pixel offset (dx, dy): exp2(-(p1^2 + p2^2)).
struct Eval {
  float dx, dy, p1, p2, G, alpha;
};

// Gaussian and alpha at offset (dx, dy) from the projected mean
__device__ __forceinline__ void evaluate_at(const float4& w1, Eval& e) {
  e.p1 = fmaf(w1.x, e.dx, w1.y * e.dy);
  e.p2 = w1.z * e.dy;
  e.G = __builtin_amdgcn_exp2f(-fmaf(e.p1, e.p1, e.p2 * e.p2));
  e.alpha = fminf(kAlphaMax, w1.w * e.G);
}

// Evaluation at pixel (fi, fj) of a record with footprint f = (i0, j0, i1 - i0,
// j1 - j0), all as floats, du = u - i0 - 1/2 and dv likewise; true if the
// footprint holds the pixel.  fi - i0 is exact (integers below 2^24), so dx has
// one rounding, and the footprint test is one unsigned compare of float bits per
// axis (a non-negative float's bits grow with its value; a negative difference
// has the sign bit set and fails).
__device__ __forceinline__ bool evaluate_f(float fi, float fj, const float4& f, float du, float dv,
                                           const float4& w1, Eval& e) {
  const float fdi = fi - f.x, fdj = fj - f.y;
  e.dx = fdi - du;
  e.dy = fdj - dv;
  evaluate_at(w1, e);
  return (__float_as_uint(fdi) <= __float_as_uint(f.z)) & (__float_as_uint(fdj) <= __float_as_uint(f.w));
}

// Lane -> pixel map of the tile kernels: the tile is cut into 8x8 pixel
// blocks, one per wave (wave w is block (w mod TW/8, w div TW/8)); each block
// is cut into groups of GW x GH pixels, numbered row-major over the block;
// lanes [g*GW*GH, (g+1)*GW*GH) hold group g and lane l is pixel (r mod GW,
// r div GW) of it (r = l mod GW*GH).  Each group walks its own list of records
// (below), so a small footprint costs one group's step, not the wave's.
template <int TW, int TH, int GW, int GH>
struct LaneMap {
  static_assert(TW % 8 == 0 && TH % 8 == 0, "tiles are whole 8x8 blocks");
  static_assert(8 % GW == 0 && 8 % GH == 0, "groups tile the 8x8 block");
  static constexpr int kGroups = 64 / (GW * GH);
  int i, j;    // this lane's pixel
  int x0, y0;  // first pixel of the wave's block
  int g;       // this lane's group
  __device__ __forceinline__ LaneMap(int txi, int tyi, int wid, int lane = (int)(threadIdx.x & 63)) {
    x0 = txi * TW + (wid % (TW / 8)) * 8;
    y0 = tyi * TH + (wid / (TW / 8)) * 8;
    g = lane / (GW * GH);
    const int r = lane % (GW * GH);
    i = x0 + (g % (8 / GW)) * GW + r % GW;
    j = y0 + (g / (8 / GW)) * GH + r / GW;
  }
};

// Group list stride: BATCH bytes plus one dword, so the lists a wave reads
// side by side start in different LDS banks.
template <int BATCH>
constexpr int kListStride = BATCH + 4;

__device__ __forceinline__ float4 footprint_floats(const float4& w0) {
  const uint32_t px = __float_as_uint(w0.z), py = __float_as_uint(w0.w);
  return make_float4((float)(px & 0xFFFFu), (float)(py & 0xFFFFu), (float)(px >> 16), (float)(py >> 16));
}

// All entries of a wave's group lists to BATCH - 1, the place of a null record
// (opacity 0: never blended) after the records of a round, so a group whose list is
// shorter than the wave's longest walks the null record instead of testing its
// position against its count at each entry (16-byte stores; the lists of a wave are
// contiguous).
template <int BATCH, int GROUPS>
__device__ __forceinline__ void clear_lists(uint8_t (*list)[kListStride<BATCH>]) {
  constexpr uint32_t kFill = 0x01010101u * (uint32_t)(BATCH - 1);
  static_assert(GROUPS * kListStride<BATCH> % 16 == 0, "whole 16-byte words");
  uint4* p = reinterpret_cast<uint4*>(&list[0][0]);
  for (int k = threadIdx.x & 63; k < GROUPS * kListStride<BATCH> / 16; k += 64)
    p[k] = make_uint4(kFill, kFill, kFill, kFill);
}

// Per-group lists: list[g][0 .. count) receives, in ascending (= depth) order, the
// staged records that may contribute to a pixel of group g of the wave's block.
__device__ __forceinline__ void append_if(bool h, uint8_t* list, int& c, int k) {
  const uint64_t m = __ballot(h);
  if (h) list[c + (int)lanemask_lt_count(m)] = (uint8_t)k;
  c += (int)__popcll(m);
}

// Largest exponent Q = p1^2 + p2^2 at which a record of this opacity can reach
// the alpha threshold: opac * exp2(-Q) >= 1/255 <=> Q <= log2(255 opac).  The
// slack (0.7 % in alpha) covers the rounding of the logarithm here and of Q and
// exp2 in evaluate_at.
__device__ __forceinline__ float q_limit(float opac) { return __builtin_amdgcn_logf(255.0f * opac) + 0.01f; }

// Whether a staged record may contribute to a group: its footprint rectangle
// meets the group, and the smallest Q over the group can stay within q_limit.
// Q = p1^2 + p2^2 with p1 = ca dx + cb dy and p2 = cc dy, both linear, so over a
// GW x GH group |p1| is at least its value at the centre less its half range
// (|ca| (GW-1) + |cb| (GH-1)) / 2, and likewise p2; the sum of the two squared
// minima bounds Q from below.  Every pixel of a group rejected here has
// alpha < 1/255 (the compositing skips such entries), so the result is the same
// bit for bit.  The margins cover the rounding of this estimate (a few ulp of
// the summed terms, FP32) hundreds of times over; a NaN keeps the record.
struct GroupTest {
  float i0, i1, j0, j1;  // footprint relative to the first group's first pixel
  float p1, m1, sx, sy;  // p1 at the centre of the first group, half range, steps per pixel
  float p2, m2, sy2;
  float q;
  // f, du, dv: as for evaluate_f; (x0, y0): first pixel of the first group; the groups tested lie
  // within 32 pixels of it
  template <int GW, int GH>
  __device__ __forceinline__ void load(const float4& f, float du, float dv, const float4& w1, float q_lim, int x0,
                                       int y0) {
    i0 = f.x - (float)x0, i1 = i0 + f.z;
    j0 = f.y - (float)y0, j1 = j0 + f.w;
    q = q_lim;
    const float dx = (0.5f * (GW - 1) - i0) - du;
    const float dy = (0.5f * (GH - 1) - j0) - dv;
    sx = w1.x, sy = w1.y, sy2 = w1.z;
    p1 = fmaf(sx, dx, sy * dy);
    p2 = sy2 * dy;
    const float ax = fabsf(sx), ay = fabsf(sy), a2 = fabsf(sy2);
    const float ex = fabsf(dx) + 32.0f, ey = fabsf(dy) + 32.0f;  // largest offsets tested
    m1 = fmaf(0.5f * (GW - 1), ax, fmaf(0.5f * (GH - 1), ay, fmaf(1e-5f, fmaf(ax, ex, ay * ey), 1e-3f)));
    m2 = fmaf(0.5f * (GH - 1), a2, fmaf(1e-5f, a2 * ey, 1e-3f));
  }
  // the footprint meets the group whose first pixel is (c, r) from (x0, y0)
  template <int GW, int GH>
  __device__ __forceinline__ bool meets(float c, float r) const {
    return (i0 <= c + (GW - 1)) & (i1 >= c) & (j0 <= r + (GH - 1)) & (j1 >= r);
  }
  // squared lower bound of |p2| over the groups of row r
  __device__ __forceinline__ float row(float r) const {
    const float a = fmaxf(fabsf(fmaf(sy2, r, p2)) - m2, 0.0f);
    return a * a;
  }
  __device__ __forceinline__ bool reach(float c, float r, float row2) const {
    const float a = fmaxf(fabsf(fmaf(sx, c, fmaf(sy, r, p1))) - m1, 0.0f);
    return !(fmaf(a, a, row2) > q);
  }
};

// First step of a wave's lists: the staged records whose footprint meets the
// wave's 8x8 block (about two in five of a 16x16 tile's), so the per-group tests
// run on full lanes of candidates only.
template <int BATCH>
__device__ __forceinline__ int wave_candidates(const float4* s_w0, int nb, int x0, int y0, uint8_t* cand) {
  static_assert(BATCH <= 256, "record indices are bytes");
  const int lane = threadIdx.x & 63;
  int c = 0;
  for (int base = 0; base < nb; base += 64) {
    const int k = base + lane;
    bool h = false;
    if (k < nb) {
      const uint32_t px = __float_as_uint(s_w0[k].z), py = __float_as_uint(s_w0[k].w);
      const int i0 = (int)(px & 0xFFFFu), j0 = (int)(py & 0xFFFFu);
      h = i0 <= x0 + 7 && i0 + (int)(px >> 16) >= x0 && j0 <= y0 + 7 && j0 + (int)(py >> 16) >= y0;
    }
    append_if(h, cand, c, k);
  }
  return c;
}

// 4x2 groups (two columns of four pixels, four rows of two; row-major).  s_w0[k].y
// holds q_limit of the record (its view is not needed once staged).  Returns the
// length of the longest list.
template <int BATCH>
__device__ __forceinline__ int wave_compact8(const float4* s_w0, const float4* s_f, const float4* s_w1,
                                                 const float4* s_w2, int nb, int x0, int y0, uint8_t* cand,
                                                 uint8_t (*list)[kListStride<BATCH>]) {
  const int lane = threadIdx.x & 63;
  const int nc = wave_candidates<BATCH>(s_w0, nb, x0, y0, cand);
  int c0 = 0, c1 = 0, c2 = 0, c3 = 0, c4 = 0, c5 = 0, c6 = 0, c7 = 0;
  for (int base = 0; base < nc; base += 64) {
    const bool in = base + lane < nc;
    const int k = in ? (int)cand[base + lane] : 0;
    const float4 w0 = s_w0[k];
    GroupTest t;
    t.load<4, 2>(s_f[k], w0.x, s_w2[k].w, s_w1[k], w0.y, x0, y0);
    const bool xa = in & (t.i0 <= 3.0f), xb = in & (t.i1 >= 4.0f);  // a candidate meets the block
    auto rows = [&](float r, uint8_t* la, int& ca, uint8_t* lb, int& cb) {
      const bool y = (t.j0 <= r + 1.0f) & (t.j1 >= r);
      const float r2 = t.row(r);
      append_if(xa & y & t.reach(0.0f, r, r2), la, ca, k);
      append_if(xb & y & t.reach(4.0f, r, r2), lb, cb, k);
    };
    rows(0.0f, list[0], c0, list[1], c1);
    rows(2.0f, list[2], c2, list[3], c3);
    rows(4.0f, list[4], c4, list[5], c5);
    rows(6.0f, list[6], c6, list[7], c7);
  }
  return max(max(max(c0, c1), max(c2, c3)), max(max(c4, c5), max(c6, c7)));
}

struct TileArgs {
  const Record* records;
  const uint32_t* pair_records;
  const uint32_t* ranges;
  int W, H, tiles_x_n, tiles_per_view;
  int64_t n_tiles;
};

// Work distribution shared by the tile kernels: either one work-group per tile
// (queue == nullptr) or persistent work-groups taking tiles from the device
// queue built by bin_sort, longest lists first.
//
// Every work-group ends on exactly one fetch past the end, so those fetches
// return n_tiles .. n_tiles + gridDim.x - 1; the work-group that draws the last
// of them knows no other will read the head again and puts it back to zero.
// A second launch on the same sorted frame (a repeated forward, a second
// backward) therefore walks the whole queue again.
template <class Body>
__device__ __forceinline__ void for_each_tile(const TileArgs& t, uint32_t* queue, int head, Body body) {
  if (queue == nullptr) {
    body((int)blockIdx.x);
    return;
  }
  __shared__ uint32_t s_next;
  for (;;) {
    if (threadIdx.x == 0) s_next = atomicAdd(&queue[head], 1u);
    __syncthreads();
    const uint32_t k = s_next;
    __syncthreads();
    if ((int64_t)k >= t.n_tiles) {
      if (threadIdx.x == 0 && (int64_t)k == t.n_tiles + (int64_t)gridDim.x - 1) atomicExch(&queue[head], 0u);
      break;
    }
    body((int)queue[2 + k]);
  }
}

// Persistent grid for the queue mode: enough work-groups to fill every CU a few times over.
inline dim3 tile_grid(int64_t n_tiles, bool queued) {
  const int64_t cap = 256 * 8;
  return dim3((unsigned)(queued ? (n_tiles < cap ? (n_tiles > 0 ? n_tiles : 1) : cap) : n_tiles));
}

inline bool batch_supported(int b) { return b == 64 || b == 128 || b == 256; }

}  // namespace
}  // namespace gs
