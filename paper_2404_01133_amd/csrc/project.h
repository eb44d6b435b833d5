// FP64 projection of one Gaussian (the "proj" operator of Eq. 1, Sec. 3.1,
// following 3DGS), shared by the forward preprocess and its adjoint.  Every
// translation unit that includes this header is compiled with
// -ffp-contract=off: the operation order below is the reproducibility contract
// for culls, footprints and depth keys.
#pragma once

#include "gs_common.h"

namespace gs {

constexpr int kMaxLevels = 8;

struct LevelPtrs {
  const float* means;
  const void* scales;
  const void* quats;
  const void* opac;
  const void* sh;
  int64_t n;
  int sh_deg;  // SH bands stored
  bool half;   // attributes other than the centre are binary16
};

__host__ __forceinline__ LevelPtrs level_ptrs(const gs_gaussians& g) {
  return LevelPtrs{g.means, g.scales, g.quats, g.opac, g.sh, g.n, g.sh_degree, g.attr_half != 0};
}

// attribute i of an array stored as FP32 or binary16 (widening is exact); the
// storage is a template parameter so each record's code has no per-load branch
template <bool HALF>
__device__ __forceinline__ float attr(const void* p, int64_t i) {
  if constexpr (HALF) return (float)reinterpret_cast<const _Float16*>(p)[i];
  else return reinterpret_cast<const float*>(p)[i];
}

__device__ __forceinline__ double dmin_(double a, double b) { return b < a ? b : a; }
__device__ __forceinline__ double dmax_(double a, double b) { return a < b ? b : a; }

// index of the (view, block) segment holding record g: largest p with offsets[p] <= g
__device__ __forceinline__ int find_segment(const int64_t* __restrict__ offsets, int nseg, int64_t g) {
  int lo = 0, hi = nseg;  // invariant: offsets[lo] <= g < offsets[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (offsets[mid] <= g) lo = mid; else hi = mid;
  }
  return lo;
}

// Normalisation constants of the real SH basis up to degree 3 (m = -l..l,
// Condon-Shortley phase kept), evaluated at a unit direction below.
constexpr double kSH00 = 0.28209479177387814;
constexpr double kSH1 = 0.4886025119029199;
constexpr double kSH2a = 1.0925484305920792;
constexpr double kSH2b = 0.31539156525252005;
constexpr double kSH2c = 0.5462742152960396;
constexpr double kSH3a = 0.5900435899266435;
constexpr double kSH3b = 2.890611442640554;
constexpr double kSH3c = 0.4570457994644658;
constexpr double kSH3d = 0.3731763325901154;
constexpr double kSH3e = 1.445305721320277;

// Colour sum_k Y_k f_k (per channel, k ascending) with the basis terms of
// sh_basis computed one at a time, so no basis array is live.  coef(i):
// coefficient plane i of the bands up to deg.
template <class Coef>
__device__ __forceinline__ void sh_colour(double x, double y, double z, int deg, Coef coef, double col[3]) {
  auto term = [&](int k, double Yk) {
#pragma unroll
    for (int ch = 0; ch < 3; ++ch) col[ch] += Yk * (double)coef(3 * k + ch);
  };
  term(0, kSH00);
  if (deg < 1) return;
  term(1, -kSH1 * y);
  term(2, kSH1 * z);
  term(3, -kSH1 * x);
  if (deg < 2) return;
  const double xx = x * x, yy = y * y, zz = z * z;
  term(4, kSH2a * (x * y));
  term(5, -kSH2a * (y * z));
  term(6, kSH2b * (2.0 * zz - xx - yy));
  term(7, -kSH2a * (x * z));
  term(8, kSH2c * (xx - yy));
  if (deg < 3) return;
  term(9, -kSH3a * (y * (3.0 * xx - yy)));
  term(10, kSH3b * (x * y * z));
  term(11, -kSH3c * (y * (4.0 * zz - xx - yy)));
  term(12, kSH3d * (z * (2.0 * zz - 3.0 * xx - 3.0 * yy)));
  term(13, -kSH3c * (x * (4.0 * zz - xx - yy)));
  term(14, kSH3e * (z * (xx - yy)));
  term(15, -kSH3a * (x * (xx - 3.0 * yy)));
}

// Coefficient planes of the bands up to deg, 0 beyond (one branch per band: a branch per load makes the
// loads wait for each other)
template <bool HALF>
__device__ __forceinline__ void load_sh(const LevelPtrs& L, int64_t gi, int deg, float (&f)[48]) {
  auto load = [&](int i) { f[i] = attr<HALF>(L.sh, (int64_t)i * L.n + gi); };
#pragma unroll
  for (int i = 0; i < 48; ++i) f[i] = 0.0f;
#pragma unroll
  for (int i = 0; i < 3; ++i) load(i);
  if (deg >= 1) {
#pragma unroll
    for (int i = 3; i < 12; ++i) load(i);
  }
  if (deg >= 2) {
#pragma unroll
    for (int i = 12; i < 27; ++i) load(i);
  }
  if (deg >= 3) {
#pragma unroll
    for (int i = 27; i < 48; ++i) load(i);
  }
}

// Camera centre C = -R^T t.
__device__ __forceinline__ void camera_centre(const gs_camera& cam, double C[3]) {
  const double* R = cam.R;
  C[0] = -((R[0] * cam.t[0] + R[3] * cam.t[1]) + R[6] * cam.t[2]);
  C[1] = -((R[1] * cam.t[0] + R[4] * cam.t[1]) + R[7] * cam.t[2]);
  C[2] = -((R[2] * cam.t[0] + R[5] * cam.t[1]) + R[8] * cam.t[2]);
}

// Camera v, the same v in the whole wave, through the scalar cache: it then takes no vector registers
// (the cameras are read-only for the kernel, which is what the constant address space says).
__device__ __forceinline__ gs_camera uniform_camera(const gs_camera* cams, int v) {
  const auto* p = (const __attribute__((address_space(4))) gs_camera*)cams + v;
  gs_camera c;
#pragma unroll
  for (int k = 0; k < 9; ++k) c.R[k] = p->R[k];
#pragma unroll
  for (int k = 0; k < 3; ++k) c.t[k] = p->t[k];
  c.fx = p->fx;
  c.fy = p->fy;
  c.cx = p->cx;
  c.cy = p->cy;
  c.znear = p->znear;
  return c;
}

// f(key) with the key in a scalar register, once for each key among the wave's active lanes (with
// the lanes that have it active).  Used for view and level, which almost always are one for the whole
// wave: the camera and the level's pointers are then scalar.  The loop's condition is the wave's, not a
// lane's: lanes that left the loop one by one would run f after it, all together, with one lane's key.
template <class F>
__device__ __forceinline__ void for_each_key(int key, F f) {
  for (uint64_t left = __ballot(1); left;) {
    const int u = __builtin_amdgcn_readlane(key, __builtin_ctzll(left));
    const bool mine = key == u;
    if (mine) f(__builtin_amdgcn_readfirstlane(key));
    left &= ~__ballot(mine);
  }
}

// What the projection needs of a view in FP64 and is the same for every record.  A work-group keeps
// them in LDS for up to kLdsViews views (15 FP64 operations and two divisions less per record).
struct ViewConst {
  double C[3], limx, limy;  // camera centre; guard-band limits of x/z and y/z
  __device__ __forceinline__ void load(const gs_camera& cam, int W, int H) {
    camera_centre(cam, C);
    limx = 1.3 * ((0.5 * W) / cam.fx);
    limy = 1.3 * ((0.5 * H) / cam.fy);
  }
};
constexpr int kLdsViews = 32;

__device__ __forceinline__ void load_views(const gs_camera* cams, int V, int W, int H, ViewConst (&s_view)[kLdsViews]) {
  if ((int)threadIdx.x < V && threadIdx.x < kLdsViews) s_view[threadIdx.x].load(cams[threadIdx.x], W, H);
}
__device__ __forceinline__ ViewConst view_const(const gs_camera* cams, int V, int W, int H,
                                                const ViewConst (&s_view)[kLdsViews], int v) {
  if (V <= kLdsViews) return s_view[v];
  ViewConst c;
  c.load(cams[v], W, H);
  return c;
}

// Stored geometry of one Gaussian, and the part of the projection that no view enters.
struct Shape {
  float m[3], s[3], q[4], op;
  double Lm[3][3];  // Rq diag(s)
  template <bool HALF>
  __device__ __forceinline__ void load(const LevelPtrs& L, int64_t gi) {
#pragma unroll
    for (int k = 0; k < 3; ++k) m[k] = L.means[k * L.n + gi];
    op = attr<HALF>(L.opac, gi);
#pragma unroll
    for (int k = 0; k < 3; ++k) s[k] = attr<HALF>(L.scales, k * L.n + gi);
  }
  template <bool HALF>
  __device__ __forceinline__ void load_rotation(const LevelPtrs& L, int64_t gi) {
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = attr<HALF>(L.quats, k * L.n + gi);
  }
  // false: no rotation (zero, non-finite or overflowing quaternion), the Gaussian is culled
  __device__ __forceinline__ bool rotate() {
    const double q0 = q[0], q1 = q[1], q2 = q[2], q3 = q[3];
    const double qn2 = ((q0 * q0 + q1 * q1) + q2 * q2) + q3 * q3;
    if (!(qn2 > 0.0 && qn2 <= 1.0e300)) return false;
    const double qinv = 1.0 / sqrt(qn2);
    const double w = q0 * qinv, x = q1 * qinv, y = q2 * qinv, z = q3 * qinv;
    double Rq[3][3];
    Rq[0][0] = 1.0 - 2.0 * (y * y + z * z);
    Rq[0][1] = 2.0 * (x * y - w * z);
    Rq[0][2] = 2.0 * (x * z + w * y);
    Rq[1][0] = 2.0 * (x * y + w * z);
    Rq[1][1] = 1.0 - 2.0 * (x * x + z * z);
    Rq[1][2] = 2.0 * (y * z - w * x);
    Rq[2][0] = 2.0 * (x * z - w * y);
    Rq[2][1] = 2.0 * (y * z + w * x);
    Rq[2][2] = 1.0 - 2.0 * (x * x + y * y);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) Lm[i][j] = Rq[i][j] * (double)s[j];
    return true;
  }
};

// What the forward projection hands on for one Gaussian in one view.
struct Geo {
  double rz, ux, uy;  // 1/tz, tx/tz, ty/tz in camera space
  double u, v;
  double b, c, det;   // of the dilated 2D covariance [[a, b], [b, c]]
  float depth;
  int i0, i1, j0, j1;
};

// Culling and footprint in two parts.  project_front needs centre, scale and opacity (28 B), which decide
// most culls — the near plane, the opacity threshold, and a footprint that certainly misses the image
// (below); project_back needs the rotation (16 B) too.  The SH coefficients are read only for survivors.
//
// Early footprint test: the projected covariance is J W Rq diag(s)^2 Rq^T W^T J^T
// with W and Rq rotations, so its trace is at most |J|_F^2 s_max^2, and the
// larger eigenvalue of the dilated matrix is below that trace + 0.6.  With |J|_F^2
// bounded through the guard-band limits of x/z and y/z, 3 sqrt(bound) + 2 px is
// more than the radius ceil(3 sqrt(lmax)) computed below (the relative slack of
// 1e-6 covers the rounding of both sides), and u, v are computed by the same
// operations as below, so a centre farther than that outside the image is one
// the exact test would cull too.  Non-finite values fail every comparison and
// take the exact path.
__device__ __forceinline__ bool project_front(const Shape& g, const gs_camera& cam, const ViewConst& vc, int W, int H,
                                              Geo& o) {
  const double* R = cam.R;
  const double m0 = g.m[0], m1 = g.m[1], m2 = g.m[2];
  const double tx = ((R[0] * m0 + R[1] * m1) + R[2] * m2) + cam.t[0];
  const double ty = ((R[3] * m0 + R[4] * m1) + R[5] * m2) + cam.t[1];
  const double tz = ((R[6] * m0 + R[7] * m1) + R[8] * m2) + cam.t[2];
  if (!(tz > cam.znear)) return false;
  if (!((double)g.op >= 1.0 / 255.0)) return false;
  o.depth = (float)tz;
  o.rz = 1.0 / tz;
  o.ux = tx * o.rz;
  o.uy = ty * o.rz;
  o.u = cam.fx * o.ux + cam.cx;
  o.v = cam.fy * o.uy + cam.cy;
  const double smax = dmax_(fabs((double)g.s[0]), dmax_(fabs((double)g.s[1]), fabs((double)g.s[2])));
  const double jx = cam.fx * o.rz, jy = cam.fy * o.rz;
  const double jf2 = jx * jx * (1.0 + vc.limx * vc.limx) + jy * jy * (1.0 + vc.limy * vc.limy);
  const double rb = 3.0 * sqrt((jf2 * (smax * smax) + 0.6) * (1.0 + 1e-6)) + 2.0;
  return !((o.u + rb) - 0.5 < 0.0 || (o.u - rb) - 0.5 > (double)(W - 1) || (o.v + rb) - 0.5 < 0.0 ||
           (o.v - rb) - 0.5 > (double)(H - 1));
}

__device__ __forceinline__ bool project_back(const Shape& g, const gs_camera& cam, const ViewConst& vc, int W, int H,
                                             Geo& o) {
  const double* R = cam.R;
  double WL[3][3];  // R_cam Lm
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int j = 0; j < 3; ++j)
      WL[i][j] = (R[3 * i + 0] * g.Lm[0][j] + R[3 * i + 1] * g.Lm[1][j]) + R[3 * i + 2] * g.Lm[2][j];
  const double uxc = dmin_(vc.limx, dmax_(-vc.limx, o.ux));
  const double uyc = dmin_(vc.limy, dmax_(-vc.limy, o.uy));
  const double J00 = cam.fx * o.rz, J02 = -(cam.fx * uxc) * o.rz;
  const double J11 = cam.fy * o.rz, J12 = -(cam.fy * uyc) * o.rz;
  double M[2][3];  // J WL
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    M[0][j] = J00 * WL[0][j] + J02 * WL[2][j];
    M[1][j] = J11 * WL[1][j] + J12 * WL[2][j];
  }
  const double n0 = (M[0][0] * M[0][0] + M[0][1] * M[0][1]) + M[0][2] * M[0][2];
  const double n1 = (M[1][0] * M[1][0] + M[1][1] * M[1][1]) + M[1][2] * M[1][2];
  o.b = (M[0][0] * M[1][0] + M[0][1] * M[1][1]) + M[0][2] * M[1][2];
  const double a = n0 + 0.3;
  o.c = n1 + 0.3;
  const double cr0 = M[0][1] * M[1][2] - M[0][2] * M[1][1];
  const double cr1 = M[0][2] * M[1][0] - M[0][0] * M[1][2];
  const double cr2 = M[0][0] * M[1][1] - M[0][1] * M[1][0];
  o.det = (((cr0 * cr0 + cr1 * cr1) + cr2 * cr2) + 0.3 * (n0 + n1)) + 0.09;
  if (!(o.det > 0.0 && o.det <= 1.0e300)) return false;
  const double hd = 0.5 * (a - o.c);
  const double lmax = 0.5 * (a + o.c) + sqrt(hd * hd + o.b * o.b);
  if (!(lmax <= 1.0e300)) return false;
  const double r = ceil(3.0 * sqrt(lmax));
  const double i0 = dmax_(0.0, ceil((o.u - r) - 0.5));
  const double i1 = dmin_((double)(W - 1), floor((o.u + r) - 0.5));
  const double j0 = dmax_(0.0, ceil((o.v - r) - 0.5));
  const double j1 = dmin_((double)(H - 1), floor((o.v + r) - 0.5));
  if (!(i0 <= i1) || !(j0 <= j1)) return false;
  o.i0 = (int)i0;
  o.i1 = (int)i1;
  o.j0 = (int)j0;
  o.j1 = (int)j1;
  return true;
}

// sqrt(log2(e) / 2): the conic factor is scaled so the Gaussian is exp2(-Q).
constexpr double kConicScale = 0.84932180028801907;

}  // namespace gs
