// Entry points of the row kernels: small systems, one launch per evaluation or step.
#include "rows_launch.h"

namespace nb {
namespace {

template <class Epi>
int rows(RowEval e, const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi) {
  return c.precision == NBODY_FP64 ? rows64(e, c, x, w, u, epi) : rows32(e, c, x, w, u, epi);
}

}  // namespace

int launch_rows_accel(const RowCall& c, const double* x, double* a) {
  return rows(RowEval::kAccel, c, x, nullptr, nullptr, EpiStore{c.G, a, nullptr, nullptr});
}

int launch_rows_jerk(const RowCall& c, const double* x, const double* v, double* a, double* jk) {
  return rows(RowEval::kJerk, c, x, v, nullptr, EpiStore{c.G, a, jk, nullptr});
}

int launch_rows_snap(const RowCall& c, const double* x, const double* v, const double* acc, double* a, double* jk,
                     double* sn) {
  return rows(RowEval::kSnap, c, x, v, acc, EpiStore{c.G, a, jk, sn});
}

int launch_rows_vjp(const RowCall& c, const double* x, const double* w, double* gx, double* gm) {
  return rows(RowEval::kVjp, c, x, w, nullptr, EpiStore{c.G, gx, gm, nullptr});
}

int launch_rows_potential(const RowCall& c, const double* x, double scale, double* phi) {
  return rows64(RowEval::kPot, c, x, nullptr, nullptr, EpiStore{scale, phi, nullptr, nullptr});
}

int launch_rows_kdk(const RowCall& c, const double* x, double* xo, double* v, double* a, double h, double dt, int nkicks) {
  return rows(RowEval::kAccel, c, x, nullptr, nullptr, EpiKdk{c.G, h, dt, nkicks, x, xo, v, a});
}

int launch_rows_hermite4(const RowCall& c, const double* xp, const double* vp, double* x, double* v, double* a,
                         double* jk, double* xo, double* vo, double dt) {
  return rows(RowEval::kJerk, c, xp, vp, nullptr, EpiHermite4{c.G, dt, x, v, a, jk, xo, vo});
}

int launch_rows_hermite6(const RowCall& c, double* const* p, double* x, double* v, double* a, double* jk, double* sn,
                         double* cr, double* const* o, double dt) {
  const EpiHermite6 epi{c.G, dt, x, v, a, jk, sn, cr, o ? o[0] : nullptr, o ? o[1] : nullptr, o ? o[2] : nullptr};
  return rows(RowEval::kSnap, c, p[0], p[1], p[2], epi);
}

int launch_rows_adjoint(const RowCall& c, const double* x, const double* lv, double* lx, double* gm, double* lvo,
                        double dt) {
  return rows(RowEval::kVjp, c, x, lv, nullptr, EpiAdjoint{c.G, dt, lx, gm, lv, lvo});
}

}  // namespace nb
