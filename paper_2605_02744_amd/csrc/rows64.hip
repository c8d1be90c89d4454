// The FP64 row kernels (rows64.h), one launch for each evaluation and update.
#include "rows64.h"
#include "rows_launch.h"

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
int launch(const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi) {
  if (c.n == 0) return NBODY_OK;
  if (c.n > kRowsMaxN) return set_error(NBODY_EINVAL, "row kernel: n too large");
  const RowArgs A{(int)c.n, x, c.m, w, u, c.eps * c.eps};
  if (c.n <= kAheadMaxN) return launch_u<E, (E::NW > 7 ? 2 : 4)>(A, c.excl, epi, c.s);
  return launch_u<E, 1>(A, c.excl, epi, c.s);
}

}  // namespace

template <class Epi>
int rows64(RowEval e, const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi) {
  if constexpr (Epi::eval == RowEval::kAny) {
    switch (e) {
      case RowEval::kAccel: return launch<RowAccel>(c, x, w, u, epi);
      case RowEval::kJerk: return launch<RowJerk>(c, x, w, u, epi);
      case RowEval::kSnap: return launch<RowSnap>(c, x, w, u, epi);
      case RowEval::kVjp: return launch<RowVjp>(c, x, w, u, epi);
      case RowEval::kPot: return launch<RowPot>(c, x, w, u, epi);
      default: return set_error(NBODY_EINVAL, "row kernel: unknown evaluation");
    }
  } else if constexpr (Epi::eval == RowEval::kAccel) {
    return launch<RowAccel>(c, x, w, u, epi);
  } else if constexpr (Epi::eval == RowEval::kJerk) {
    return launch<RowJerk>(c, x, w, u, epi);
  } else if constexpr (Epi::eval == RowEval::kSnap) {
    return launch<RowSnap>(c, x, w, u, epi);
  } else {
    return launch<RowVjp>(c, x, w, u, epi);
  }
}

#define NB_ROWS64(Epi) \
  template int rows64<Epi>(RowEval, const RowCall&, const double*, const double*, const double*, const Epi&)
NB_ROWS64(EpiStore);
NB_ROWS64(EpiKdk);
NB_ROWS64(EpiHermite4);
NB_ROWS64(EpiHermite6);
NB_ROWS64(EpiAdjoint);

}  // namespace nb
