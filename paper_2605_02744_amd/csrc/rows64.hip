// Launchers of the FP64 row kernels (rows64.h): evaluations and whole steps of
// systems of up to kRowsMaxN particles, one launch each.
#include "rows64.h"

namespace nb {
namespace {

// Up to this many particles the records are loaded ahead (see rows64.h).
constexpr int64_t kAheadMaxN = 2048;

template <class E, int U, class Epi>
int launch_u(const RowArgs& A, bool excl, const Epi& epi, hipStream_t s) {
  const unsigned grid = (unsigned)((A.n + kRows - 1) / kRows);
  if (excl) rows64_kernel<E, U, true, Epi><<<grid, kRowT, 0, s>>>(A, epi);
  else rows64_kernel<E, U, false, Epi><<<grid, kRowT, 0, s>>>(A, epi);
  NB_LAUNCH_CHECK("rows64_kernel");
  return NBODY_OK;
}

template <class E, class Epi>
int launch(int64_t n, const double* x, const double* m, const double* w, const double* u, double eps, bool excl,
           const Epi& epi, hipStream_t s) {
  if (n == 0) return NBODY_OK;
  if (n > kRowsMaxN) return set_error(NBODY_EINVAL, "row kernel: n too large");
  const RowArgs A{(int)n, x, m, w, u, eps * eps};
  if (n <= kAheadMaxN) return launch_u<E, (E::NW > 7 ? 2 : 4)>(A, excl, epi, s);
  return launch_u<E, 1>(A, excl, epi, s);
}

}  // namespace

int launch_rows64_accel(int64_t n, const double* x, const double* m, double* a, double G, double eps, bool excl,
                        hipStream_t s) {
  return launch<RowAccel>(n, x, m, nullptr, nullptr, eps, excl, EpiStore{G, a, nullptr, nullptr}, s);
}

int launch_rows64_jerk(int64_t n, const double* x, const double* v, const double* m, double* a, double* jk, double G,
                       double eps, bool excl, hipStream_t s) {
  return launch<RowJerk>(n, x, m, v, nullptr, eps, excl, EpiStore{G, a, jk, nullptr}, s);
}

int launch_rows64_snap(int64_t n, const double* x, const double* v, const double* acc, const double* m, double* a,
                       double* jk, double* sn, double G, double eps, bool excl, hipStream_t s) {
  return launch<RowSnap>(n, x, m, v, acc, eps, excl, EpiStore{G, a, jk, sn}, s);
}

int launch_rows64_vjp(int64_t n, const double* x, const double* m, const double* w, double* gx, double* gm, double G,
                      double eps, bool excl, hipStream_t s) {
  return launch<RowVjp>(n, x, m, w, nullptr, eps, excl, EpiStore{G, gx, gm, nullptr}, s);
}

int launch_rows64_potential(int64_t n, const double* x, const double* m, double eps, double scale, double* phi,
                            hipStream_t s) {
  return launch<RowPot>(n, x, m, nullptr, nullptr, eps, true, EpiStore{scale, phi, nullptr, nullptr}, s);
}

int launch_rows64_kdk(int64_t n, const double* x, double* xo, double* v, double* a, const double* m, double h, double dt,
                      int nkicks, double G, double eps, bool excl, hipStream_t s) {
  return launch<RowAccel>(n, x, m, nullptr, nullptr, eps, excl, EpiKdk{G, h, dt, nkicks, x, xo, v, a}, s);
}

int launch_rows64_hermite4(int64_t n, const double* xp, const double* vp, const double* m, double* x, double* v,
                           double* a, double* jk, double* xo, double* vo, double dt, double G, double eps, bool excl,
                           hipStream_t s) {
  return launch<RowJerk>(n, xp, m, vp, nullptr, eps, excl, EpiHermite4{G, dt, x, v, a, jk, xo, vo}, s);
}

int launch_rows64_hermite6(int64_t n, double* const* p, const double* m, double* x, double* v, double* a, double* jk,
                           double* sn, double* cr, double* const* o, double dt, double G, double eps, bool excl,
                           hipStream_t s) {
  const EpiHermite6 epi{G, dt, x, v, a, jk, sn, cr, o ? o[0] : nullptr, o ? o[1] : nullptr, o ? o[2] : nullptr};
  return launch<RowSnap>(n, p[0], m, p[1], p[2], eps, excl, epi, s);
}

int launch_rows64_adjoint(int64_t n, const double* x, const double* m, const double* lv, double* lx, double* gm,
                          double* lvo, double dt, double G, double eps, bool excl, hipStream_t s) {
  return launch<RowVjp>(n, x, m, lv, nullptr, eps, excl, EpiAdjoint{G, dt, lx, gm, lv, lvo}, s);
}

}  // namespace nb
