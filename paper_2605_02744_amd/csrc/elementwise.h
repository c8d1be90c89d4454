// The integrators' elementwise arithmetic, shared by the O(N) kernels
// (integrate.hip) and the row kernels that end with it (rows64.h).
#pragma once

#include <hip/hip_runtime.h>

namespace nb {

// Hermite predictor: xp = x + v dt + a dt^2/2 + j dt^3/6, vp = v + a dt + j dt^2/2.
__device__ __forceinline__ void hermite4_predict(double x, double v, double a, double jk, double dt, double& xp,
                                                 double& vp) {
  const double h2 = 0.5 * dt * dt, h3 = dt * dt * dt / 6.0;
  xp = fma(jk, h3, fma(a, h2, fma(v, dt, x)));
  vp = fma(jk, h2, fma(a, dt, v));
}

// Hermite corrector, in place on (x, v, a, jk) from the evaluation (an, jn):
//   v1 = v + (a0 + a1) dt/2 + (j0 - j1) dt^2/12
//   x1 = x + (v + v1) dt/2 + (a0 - a1) dt^2/12
__device__ __forceinline__ void hermite4_correct(double& x, double& v, double& a, double& jk, double an, double jn,
                                                 double dt) {
  const double h = 0.5 * dt, h12 = dt * dt / 12.0;
  const double v1 = fma(jk - jn, h12, fma(a + an, h, v));
  x = fma(a - an, h12, fma(v + v1, h, x));
  v = v1;
  a = an;
  jk = jn;
}

// Sixth-order Hermite predictor (shared step h, crackle c from the previous step):
//   xp = x + v h + a h^2/2 + j h^3/6 + s h^4/24 + c h^5/120
//   vp = v + a h + j h^2/2 + s h^3/6 + c h^4/24
//   ap = a + j h + s h^2/2 + c h^3/6
__device__ __forceinline__ void hermite6_predict(double x, double v, double a, double jk, double sn, double cr,
                                                 double h, double& xp, double& vp, double& ap) {
  const double c2 = h * h / 2.0, c3 = h * h * h / 6.0, c4 = h * h * h * h / 24.0, c5 = h * h * h * h * h / 120.0;
  xp = fma(cr, c5, fma(sn, c4, fma(jk, c3, fma(a, c2, fma(v, h, x)))));
  vp = fma(cr, c4, fma(sn, c3, fma(jk, c2, fma(a, h, v))));
  ap = fma(cr, c3, fma(sn, c2, fma(jk, h, a)));
}

// Sixth-order Hermite corrector, in place on (x, v, a, jk, sn) from the
// evaluation (an, jn, snn) at the predicted state:
//   v1 = v + (a + a1) h/2 - (j1 - j) h^2/10 + (s + s1) h^3/120
//   x1 = x + (v + v1) h/2 - (a1 - a) h^2/10 + (j + j1) h^3/120
// and the crackle for the next predictor, the third derivative at t = h of the
// quintic through (a, j, s) at both ends: 60 A - 36 B + 9 C with
//   A = (a1 - a - j h - s h^2/2) / h^3,  B = (j1 - j - s h) / h^2,  C = (s1 - s) / h.
__device__ __forceinline__ void hermite6_correct(double& x, double& v, double& a, double& jk, double& sn, double& cr,
                                                 double an, double jn, double snn, double h) {
  const double hh = h / 2.0, h10 = h * h / 10.0, h120 = h * h * h / 120.0;
  const double v1 = fma(sn + snn, h120, fma(-(jn - jk), h10, fma(a + an, hh, v)));
  x = fma(jk + jn, h120, fma(-(an - a), h10, fma(v + v1, hh, x)));
  v = v1;
  const double A = (an - a - jk * h - sn * (h * h / 2.0)) / (h * h * h);
  const double B = (jn - jk - sn * h) / (h * h);
  const double C = (snn - sn) / h;
  cr = 60.0 * A - 36.0 * B + 9.0 * C;
  a = an;
  jk = jn;
  sn = snn;
}

}  // namespace nb
