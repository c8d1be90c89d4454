// What a row kernel (rows64.h, rows32.h) does with its finished sums: the stores
// of an evaluation, or the elementwise update of the step it belongs to.
#pragma once

#include "common.h"
#include "elementwise.h"

namespace nb {

enum class RowEval { kAny, kAccel, kJerk, kSnap, kVjp, kPot };

// Each is called by one thread per (row i, component c < NO) with tot[q] the
// row's sum of component q; n is the components' stride.  eval: the evaluation it
// follows.

// The sums times scale: components 0-2 at o0, 3-5 at o1, 6-8 at o2 (the VJP's
// component 3 is a particle array, as is the potential's only one: o1 and o0).
struct EpiStore {
  static constexpr RowEval eval = RowEval::kAny;
  double scale;
  double *o0, *o1, *o2;
  template <int NC>
  __device__ __forceinline__ void apply(int n, int i, int c, const double* tot) const {
    double* o = c < 3 ? o0 + (size_t)c * n : c < 6 ? o1 + (size_t)(c - 3) * n : o2 + (size_t)(c - 6) * n;
    o[i] = scale * tot[c];
  }
  template <int NC> static constexpr int outs() { return NC; }
};

// KDK: a, the closing half-kick (and, with two kicks, the next step's opening
// one, each rounded separately) and with xo the drift into xo, another buffer
// than the positions x this launch still reads.
struct EpiKdk {
  static constexpr RowEval eval = RowEval::kAccel;
  double scale, h, dt;
  int nkicks;
  const double* x;
  double *xo, *v, *a;
  template <int NC>
  __device__ __forceinline__ void apply(int n, int i, int c, const double* tot) const {
    const size_t e = (size_t)c * n + i;
    const double ae = scale * tot[c];
    double ve = v[e];
    for (int k = 0; k < nkicks; ++k) ve = fma(h, ae, ve);
    a[e] = ae;
    v[e] = ve;
    if (xo) xo[e] = fma(dt, ve, x[e]);
  }
  template <int NC> static constexpr int outs() { return 3; }
};

// Fourth-order Hermite: the corrector on the row's state and with xp the next
// step's prediction, into other buffers than this launch reads.
struct EpiHermite4 {
  static constexpr RowEval eval = RowEval::kJerk;
  double scale, dt;
  double *x, *v, *a, *jk, *xp, *vp;
  template <int NC>
  __device__ __forceinline__ void apply(int n, int i, int c, const double* tot) const {
    const size_t e = (size_t)c * n + i;
    const double an = scale * tot[c], jn = scale * tot[3 + c];
    double xe = x[e], ve = v[e], ae = a[e], je = jk[e];
    hermite4_correct(xe, ve, ae, je, an, jn, dt);
    x[e] = xe; v[e] = ve; a[e] = ae; jk[e] = je;
    if (xp) hermite4_predict(xe, ve, ae, je, dt, xp[e], vp[e]);
  }
  template <int NC> static constexpr int outs() { return 3; }
};

// Sixth-order Hermite, the same way.
struct EpiHermite6 {
  static constexpr RowEval eval = RowEval::kSnap;
  double scale, dt;
  double *x, *v, *a, *jk, *sn, *cr, *xp, *vp, *ap;
  template <int NC>
  __device__ __forceinline__ void apply(int n, int i, int c, const double* tot) const {
    const size_t e = (size_t)c * n + i;
    const double an = scale * tot[c], jn = scale * tot[3 + c], s1 = scale * tot[6 + c];
    double xe = x[e], ve = v[e], ae = a[e], je = jk[e], se = sn[e], ce;
    hermite6_correct(xe, ve, ae, je, se, ce, an, jn, s1, dt);
    x[e] = xe; v[e] = ve; a[e] = ae; jk[e] = je; sn[e] = se; cr[e] = ce;
    if (xp) hermite6_predict(xe, ve, ae, je, se, ce, dt, xp[e], vp[e], ap[e]);
  }
  template <int NC> static constexpr int outs() { return 3; }
};

// The adjoint's update after a VJP: lx += gx, gm += the mass term, and with lvo
// lv's drift into lvo, another buffer than the cotangents lv this launch reads.
struct EpiAdjoint {
  static constexpr RowEval eval = RowEval::kVjp;
  double scale, dt;
  double *lx, *gm;
  const double* lv;
  double* lvo;
  template <int NC>
  __device__ __forceinline__ void apply(int n, int i, int c, const double* tot) const {
    if (c == 3) {
      gm[i] += scale * tot[3];
      return;
    }
    const size_t e = (size_t)c * n + i;
    const double l = lx[e] + scale * tot[c];
    lx[e] = l;
    if (lvo) lvo[e] = fma(dt, l, lv[e]);
  }
  template <int NC> static constexpr int outs() { return NC; }
};

}  // namespace nb
