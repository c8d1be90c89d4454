// Device-side pair arithmetic shared by the all-pairs kernels (pairs.hip, the
// row kernels) and the persistent ensemble kernel (ensemble.hip).
#pragma once

#include <type_traits>

#include "common.h"

namespace nb {

enum Mode { kFP64 = NBODY_FP64, kFP32C = NBODY_FP32C, kFP32 = NBODY_FP32 };

// Knuth's TwoSum: (hi, lo) += x with the rounding error of hi + x kept in lo.
template <typename T>
__device__ __forceinline__ void fold(T& hi, T& lo, T x) {
  T s = hi + x;
  T bp = s - hi;
  T e = (hi - (s - bp)) + (x - bp);
  hi = s;
  lo += e;
}

// 1/sqrt(r2) in FP64: the hardware estimate y (about 5e-8 relative) refined in
// one step from the residual h = 1 - r2 y^2 with the binomial series
// (1 - h)^(-1/2) = 1 + h/2 + 3h^2/8 + O(h^3): y += y h (1/2 + 3h/8).  With
// |h| ~ 1e-7 the truncated term (5h^3/16) is ~1e-22, below FP64 rounding, for
// five operations where two Newton steps take eight.
__device__ __forceinline__ double rsqrt64(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double h = fma(-r2 * y, y, 1.0);
  return fma(y * h, fma(0.375, h, 0.5), y);
}

// r2^(-3/2) in FP64 from y and the residual h = 1 - r2 y^2 in one step:
// (1 - h)^(-3/2) = 1 + 3h/2 + 15h^2/8 + O(h^3), |h| ~ 1e-7: six operations where
// refining y first and cubing it takes seven, with two roundings fewer.
__device__ __forceinline__ double rsqrt64_cubed(double r2) {
  const double y = __builtin_amdgcn_rsq(r2);
  const double y2 = y * y, h = fma(-r2, y2, 1.0), y3 = y2 * y;
  return fma(y3, h * fma(1.875, h, 1.5), y3);
}

__device__ __forceinline__ float rsqrt32(float r2) { return __builtin_amdgcn_rsqf(r2); }

// Per-mode LDS record of one j-particle and its conversion from FP64.
template <int MODE> struct JRec;

template <> struct JRec<kFP64> {
  double4 p;  // x, y, z, m
  __device__ static JRec make(double x, double y, double z, double m) {
    JRec r; r.p = make_double4(x, y, z, m); return r;
  }
};
template <> struct JRec<kFP32C> {
  float4 h;   // hi parts, mass
  float4 l;   // lo parts
  __device__ static JRec make(double x, double y, double z, double m) {
    JRec r;
    float hx = (float)x, hy = (float)y, hz = (float)z;
    r.h = make_float4(hx, hy, hz, (float)m);
    r.l = make_float4((float)(x - (double)hx), (float)(y - (double)hy), (float)(z - (double)hz), 0.f);
    return r;
  }
};
template <> struct JRec<kFP32> {
  float4 h;
  __device__ static JRec make(double x, double y, double z, double m) {
    JRec r; r.h = make_float4((float)x, (float)y, (float)z, (float)m); return r;
  }
};

// Per-mode i-particle state held in registers.
template <int MODE> struct IPos;
template <> struct IPos<kFP64> {
  double x, y, z;
  __device__ void set(double a, double b, double c) { x = a; y = b; z = c; }
  __device__ void from(const JRec<kFP64>& r) { x = r.p.x; y = r.p.y; z = r.p.z; }
};
template <> struct IPos<kFP32C> {
  float hx, hy, hz, lx, ly, lz;
  __device__ void set(double a, double b, double c) {
    hx = (float)a; hy = (float)b; hz = (float)c;
    lx = (float)(a - (double)hx); ly = (float)(b - (double)hy); lz = (float)(c - (double)hz);
  }
  __device__ void from(const JRec<kFP32C>& r) {
    hx = r.h.x; hy = r.h.y; hz = r.h.z; lx = r.l.x; ly = r.l.y; lz = r.l.z;
  }
};
template <> struct IPos<kFP32> {
  float hx, hy, hz;
  __device__ void set(double a, double b, double c) { hx = (float)a; hy = (float)b; hz = (float)c; }
  __device__ void from(const JRec<kFP32>& r) { hx = r.h.x; hy = r.h.y; hz = r.h.z; }
};

template <int MODE> using Real = typename std::conditional<MODE == kFP64, double, float>::type;

// Displacement d = x_j - x_i per mode.
__device__ __forceinline__ void disp(const JRec<kFP64>& r, const IPos<kFP64>& p, double& dx, double& dy, double& dz) {
  dx = r.p.x - p.x; dy = r.p.y - p.y; dz = r.p.z - p.z;
}
__device__ __forceinline__ void disp(const JRec<kFP32C>& r, const IPos<kFP32C>& p, float& dx, float& dy, float& dz) {
  dx = (r.h.x - p.hx) + (r.l.x - p.lx);
  dy = (r.h.y - p.hy) + (r.l.y - p.ly);
  dz = (r.h.z - p.hz) + (r.l.z - p.lz);
}
// Displacement from the hi parts only (positions rounded to FP32).
__device__ __forceinline__ void disp_hi(const JRec<kFP32C>& r, const IPos<kFP32C>& p, float& dx, float& dy, float& dz) {
  dx = r.h.x - p.hx; dy = r.h.y - p.hy; dz = r.h.z - p.hz;
}
__device__ __forceinline__ void disp(const JRec<kFP32>& r, const IPos<kFP32>& p, float& dx, float& dy, float& dz) {
  dx = r.h.x - p.hx; dy = r.h.y - p.hy; dz = r.h.z - p.hz;
}
__device__ __forceinline__ double jmass(const JRec<kFP64>& r) { return r.p.w; }
__device__ __forceinline__ float jmass(const JRec<kFP32C>& r) { return r.h.w; }
__device__ __forceinline__ float jmass(const JRec<kFP32>& r) { return r.h.w; }
__device__ __forceinline__ double rsq(double r2) { return rsqrt64(r2); }
__device__ __forceinline__ float rsq(float r2) { return rsqrt32(r2); }

// Near-field repair of FP32C pairs (see accel_kernel): a pair closer than
//   d_c(i) = max(max(kNearX, kNearN n^-1/3) |x_i|_inf, kNearEps eps)
// gets a float-float displacement.  Rounding a coordinate to FP32 moves it by
// up to u |x| (u = 2^-24), which changes a pair term m_j d / |d|^3 by about
// 3 u |x| m_j / |d|^3.  The first bound keeps that below 3u / kNearX^3 of the
// pair's own term; the second keeps it below 3u / kNearN^3 of G M / |x|^2 for
// a pair of mass M / n, which matters in small systems, where one pair at the
// radius can outweigh the whole acceleration of particle i.
constexpr float kNearX = 2.0e-2f;
constexpr float kNearN = 0.5f;
constexpr float kNearEps = 2.0f;

// Error estimate of FP32C rows and the threshold of their FP64 rescue (the
// estimate and its use are described in rescue.hip): a block of terms with
// partial sum P and closest non-repaired pair at softened distance d adds
// ((1 + kEstNear |x_i|_inf / d) |P|)^2 to E_i, and the row is recomputed in
// FP64 when kEstC u |G| sqrt(E_i) > kRescueTol |a_i|.  kEstC prices the
// arithmetic of an FP32 term (a few roundings of u); kEstNear the rounding of
// both positions to FP32, about 3 sqrt(3) u (|x_i| + |x_j|) / d relative, in
// units of kEstC u.
constexpr float kEstNear = 1.5f;
constexpr double kEstC = 4.0;
constexpr double kRescueTol = 4.0e-6;
// the flag test as sqrt(E_i) * kRescueScale |G| > |a_i|
constexpr double kRescueScale = kEstC * 5.9604644775390625e-8 / kRescueTol;

// Adds one block's share to the error estimate e (see above).
__device__ __forceinline__ float est_add(float e, float px, float py, float pz, float xinf, float r2nr) {
  const float w = fmaf(kEstNear * xinf, __builtin_amdgcn_rsqf(r2nr), 1.0f);
  return fmaf(w * w, fmaf(px, px, fmaf(py, py, pz * pz)), e);
}

// Squared repair radius of lane particle i (positions given in double) in a
// system of n particles.
__device__ __forceinline__ float near_rc2(double xa, double ya, double za, double eps, int n) {
  const float fx = fmaxf(kNearX, kNearN / cbrtf((float)(n > 0 ? n : 1)));
  const float dc = fmaxf(fx * (float)fmax(fabs(xa), fmax(fabs(ya), fabs(za))), kNearEps * (float)eps);
  return dc * dc + (float)(eps * eps);
}

// Pair terms shared by the ordered evaluations of every size.
// u = m_k w_j - m_j w_k without contraction, so that u is exactly zero for j == k.
template <typename R>
__device__ __forceinline__ R cross_weight(R mk, R wj, R mj, R wk) {
#pragma clang fp contract(off)
  R a = mk * wj;
  R b = mj * wk;
  return a - b;
}

// One VJP pair term for lane particle k and record j, displacement d = x_j - x_k:
//   g += r^-3 u - 3 r^-5 (d.u) d,  gm -= r^-3 (d . w_j),  u = m_k w_j - m_j w_k.
template <typename R>
__device__ __forceinline__ R vjp_pair(R dx, R dy, R dz, R e2, R mj, R wjx, R wjy, R wjz, R mk, R wkx, R wky,
                                      R wkz, bool self, R& px, R& py, R& pz, R& pm) {
  R r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, e2)));
  R ri = rsq(r2);
  R ri2 = ri * ri;
  R r3 = ri2 * ri;
  R r5 = r3 * ri2;
  r3 = self ? R(0) : r3;
  r5 = self ? R(0) : r5;
  R ux = cross_weight(mk, wjx, mj, wkx);
  R uy = cross_weight(mk, wjy, mj, wky);
  R uz = cross_weight(mk, wjz, mj, wkz);
  R du = fma(dz, uz, fma(dy, uy, dx * ux));
  R c = R(3) * r5 * du;
  px = fma(-c, dx, fma(r3, ux, px));
  py = fma(-c, dy, fma(r3, uy, py));
  pz = fma(-c, dz, fma(r3, uz, pz));
  R dw = fma(dz, wjz, fma(dy, wjy, dx * wjx));
  pm = fma(-r3, dw, pm);
  return r2;
}

// One acceleration + jerk pair term (App. A, Algorithm 3) for displacement d =
// x_j - x_i and velocity difference w = v_j - v_i, added to pa and pj; self
// leaves the own pair out.  Returns the softened squared distance.
template <typename R>
__device__ __forceinline__ R jerk_pair(R dx, R dy, R dz, R wx, R wy, R wz, R mj, R e2, bool self, R* pa, R* pj) {
  const R r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, e2)));
  const R ri = rsq(r2);
  R ri2 = ri * ri;
  R tj = (mj * ri) * ri2;                            // t_j = p_w,j r^-3
  if (self) {
    tj = R(0);
    ri2 = R(0);
  }
  const R vr = fma(dz, wz, fma(dy, wy, dx * wx));    // v_r = r . v
  const R qq = R(-3) * ri2 * vr;                     // q = A v_r, A = -3 r^-2
  pa[0] = fma(tj, dx, pa[0]);
  pa[1] = fma(tj, dy, pa[1]);
  pa[2] = fma(tj, dz, pa[2]);
  pj[0] = fma(tj, fma(qq, dx, wx), pj[0]);
  pj[1] = fma(tj, fma(qq, dy, wy), pj[1]);
  pj[2] = fma(tj, fma(qq, dz, wz), pj[2]);
  return r2;
}

// One acceleration + jerk + snap pair term (displacement d, velocity and
// acceleration differences w and u) added to pa, pj and ps; self leaves the own
// pair out.  Returns the softened squared distance.
template <typename R>
__device__ __forceinline__ R snap_pair(const R* d, const R* w, const R* u, R mj, R e2, bool self, R* pa, R* pj,
                                       R* ps) {
  const R r2 = fma(d[2], d[2], fma(d[1], d[1], fma(d[0], d[0], e2)));
  const R ri = rsq(r2);
  R sinv = ri * ri;
  R tj = (mj * ri) * sinv;
  if (self) {
    tj = R(0);
    sinv = R(0);
  }
  const R alpha = fma(d[2], w[2], fma(d[1], w[1], d[0] * w[0])) * sinv;
  const R wwdu = fma(d[2], u[2], fma(d[1], u[1], fma(d[0], u[0], fma(w[2], w[2], fma(w[1], w[1], w[0] * w[0])))));
  const R beta = fma(wwdu, sinv, alpha * alpha);
  const R a3 = R(-3) * alpha;
  const R b3 = R(-3) * beta;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const R P0 = tj * d[c];
    const R P1 = fma(a3, P0, tj * w[c]);
    const R P2 = fma(R(2) * a3, P1, fma(b3, P0, tj * u[c]));
    pa[c] += P0;
    pj[c] += P1;
    ps[c] += P2;
  }
  return r2;
}

}  // namespace nb
