// The FP32C and FP32 row kernels (rows32.h), one launch for each evaluation and
// update.
#include <atomic>

#include "rows32.h"
#include "rows_launch.h"

namespace nb {
namespace {

// Rows per group of lanes: 16 (four blocks of j side by side in a wave) up to 4096
// particles, which spreads a small system over more CUs, 32 above, where the
// records staged for half as many rows cost more (force 14.7 / 21.6 us at 4096, 42.8
// / 36.9 at 8191; jerk 24.5 / 33.8, 84.8 / 66.0).
constexpr int64_t kRows16MaxN = 4096;
// The force takes 16 in workgroups of half the waves from 8193 to 12288 particles, where
// three half workgroups a CU take less than two whole ones (four from there on): force
// of a Plummer sphere 53.8 / 54.1 us at 9011, 67.1 / 67.9 at 11468; of one around 100,
// most of whose pairs are corrected, 147 / 179 and 201 / 229 (tile kernels 151 and 211).
constexpr int64_t kHalfMinN = 8193, kHalfMaxN = 12288;
// The force marks its close pairs in the pair loop up to here (see row32_block).
constexpr int64_t kMarkMaxN = 2048;
// LDS a workgroup may take: records of 140 KB, so that the sums fit beside them.
constexpr size_t kRow32MaxLds = size_t(140) << 10;

// One wave per 64 / I blocks of j, at most `waves` and as many as their records fit.
template <class E, int I, bool NEAR, bool SMALL, bool EXCL, bool EST, class Epi>
int launch_i(const Row32Args& A, const Epi& epi, hipStream_t s, int waves = 16) {
  constexpr int GW = 64 / I;
  constexpr int kMost = (int)(kRow32MaxLds / row32_lds<E, I, NEAR>(1));
  const int nblk = (A.n + kJBlock - 1) / kJBlock;
  const int W = std::min(std::min(waves, kMost), (nblk + GW - 1) / GW);
  const size_t lds = row32_lds<E, I, NEAR>(W);
  auto* kernel = rows32_kernel<E, I, NEAR, SMALL, EXCL, EST, Epi>;
  // more LDS than a kernel may take unasked: allowed once per kernel and device
  static std::atomic<uint64_t> asked{0};
  const int dev = current_device();
  if (lds > (size_t(64) << 10) && (dev >= 64 || !(asked.load(std::memory_order_relaxed) >> dev & 1))) {
    NB_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kRow32MaxLds));
    if (dev < 64) asked.fetch_or(uint64_t(1) << dev, std::memory_order_relaxed);
  }
  kernel<<<(unsigned)((A.n + I - 1) / I), 64 * W, lds, s>>>(A, epi);
  NB_LAUNCH_CHECK("rows32_kernel");
  return NBODY_OK;
}

template <class E, bool NEAR, bool EXCL, bool EST, class Epi>
int launch_n(const Row32Args& A, const Epi& epi, hipStream_t s) {
  if constexpr (NEAR && !E::kChoose)
    if (A.n <= kMarkMaxN) return launch_i<E, 16, NEAR, true, EXCL, EST>(A, epi, s);
  if (A.n <= kRows16MaxN) return launch_i<E, 16, NEAR, false, EXCL, EST>(A, epi, s);
  if constexpr (E::NR == 1)
    if (A.n >= kHalfMinN && A.n <= kHalfMaxN) return launch_i<E, 16, NEAR, false, EXCL, EST>(A, epi, s, 8);
  return launch_i<E, 32, NEAR, false, EXCL, EST>(A, epi, s);
}

template <class E, class Epi>
int launch(const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi) {
  if (c.n == 0) return NBODY_OK;
  if (c.n > kRowsMaxNForce32C) return set_error(NBODY_EINVAL, "row kernel: n too large");
  const Row32Args A{(int)c.n, x, c.m, w, u, c.eps, c.G};
  constexpr bool kForce = E::NR == 1;
  if (c.precision == kFP32)
    return c.excl ? launch_n<E, false, true, false>(A, epi, c.s) : launch_n<E, false, false, false>(A, epi, c.s);
  if constexpr (kForce)
    if (c.rescue)
      return c.excl ? launch_n<E, true, true, true>(A, epi, c.s) : launch_n<E, true, false, true>(A, epi, c.s);
  return c.excl ? launch_n<E, true, true, false>(A, epi, c.s) : launch_n<E, true, false, false>(A, epi, c.s);
}

}  // namespace

template <class Epi>
int rows32(RowEval e, const RowCall& c, const double* x, const double* w, const double* u, const Epi& epi) {
  if constexpr (Epi::eval == RowEval::kAny) {
    switch (e) {
      case RowEval::kAccel: return launch<Row32Accel>(c, x, w, u, epi);
      case RowEval::kJerk: return launch<Row32Jerk>(c, x, w, u, epi);
      case RowEval::kSnap: return launch<Row32Snap>(c, x, w, u, epi);
      case RowEval::kVjp: return launch<Row32Vjp>(c, x, w, u, epi);
      default: return set_error(NBODY_EINVAL, "row kernel: unknown evaluation");
    }
  } else if constexpr (Epi::eval == RowEval::kAccel) {
    return launch<Row32Accel>(c, x, w, u, epi);
  } else if constexpr (Epi::eval == RowEval::kJerk) {
    return launch<Row32Jerk>(c, x, w, u, epi);
  } else if constexpr (Epi::eval == RowEval::kSnap) {
    return launch<Row32Snap>(c, x, w, u, epi);
  } else {
    return launch<Row32Vjp>(c, x, w, u, epi);
  }
}

#define NB_ROWS32(Epi) \
  template int rows32<Epi>(RowEval, const RowCall&, const double*, const double*, const double*, const Epi&)
NB_ROWS32(EpiStore);
NB_ROWS32(EpiKdk);
NB_ROWS32(EpiHermite4);
NB_ROWS32(EpiHermite6);
NB_ROWS32(EpiAdjoint);

}  // namespace nb
