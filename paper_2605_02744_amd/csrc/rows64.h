// Row evaluations of small FP64 systems: the device side (rows64.hip launches it).
//
// One workgroup owns kRows consecutive particles (rows) and evaluates them against
// every j, so an evaluation is one launch that leaves finished sums and needs no
// scratch; what follows an evaluation elementwise (kicks and drift, the Hermite
// corrector and predictor, the adjoint's update) is done on those sums by the
// same launch.  The tile kernels of pairs.hip split the j-range of a small
// system over workgroups instead, which costs a second kernel for the slice sums
// and a third for the update.
//
// The lanes split j (lane t takes j = t, t + 256, ...), the rows sit in scalar
// registers: a j-record loaded once serves kRows independent pairs, which hide
// the FP64 latencies of one another at the low occupancy a small system leaves,
// and neighbouring lanes load neighbouring records, straight from L2 (no LDS
// staging, no barrier in the loop).  The kRows * NC sums of a lane are added over
// four lanes of the wave by exchanging halves (each exchange sums two values at
// once), then 4 to 16 lanes add the 64 partial sums of a value with TwoSum
// (block_sums): fixed order, no atomics.  What is added plainly, at most kRowsMaxN /
// 256 = 32 terms of a lane and four lanes, is no more than a fold block of the tile
// kernels; all above is compensated as it is there.  Relative rms errors against
// extended precision, tile kernels / plain sums throughout / these: potential of 8191
// particles 5.2e-17 / 8.1e-17 / 4.9e-17, force of 5000 9.0e-17 / 9.5e-17 / 6.7e-17, of
// 1000 1.4e-16 / 1.1e-16 / 7.4e-17.  They cost up to 1 % of the longer
// launches and up to 4 % of the shorter ones (KDK step at 1024 4.69 -> 4.73 us, at 2048
// 6.8 -> 7.0, force at 5000 20.2 -> 20.5, fourth-order step there 36.6 -> 36.9).
//
// Bound: up to ~2000 particles the latency of one launch and one lane's chain
// (3.4 us per evaluation at 1000), above that FP64 issue.  Measured per step,
// tile kernels with their slice sums and updates -> rows: KDK 15.1 -> 4.5 us at
// 1024; fourth-order Hermite 58 -> 36 us at 5000.  Rows per workgroup, accel /
// jerk / snap / vjp in us: at 1024 4 rows 3.4 / 4.6 / 6.0 / 4.5, 2 rows 3.4 / 4.9 /
// 5.5 / 4.7, 8 rows 4.3 / 7.0 / - / 7.5 (half the CUs idle); at 5000 4 rows 20.6 /
// 35 / 61 / 39, 2 rows 28 / 47 / 68 / 51 (record loads), 6 rows 23 / 39 / - / 46
// (fewer workgroups than the CUs divide evenly).  Up to 2048 particles a lane
// loads its records four ahead (snap: two): right after the launch that wrote
// them they come from beyond L2, and with one or two waves per SIMD nothing else
// hides that (KDK step at 1024 5.2 us one at a time, 4.5 us four ahead); above,
// other waves do, and fewer registers are worth more.
#pragma once

#include "pair_math.h"
#include "row_update.h"
#include "wave64.h"

namespace nb {
namespace {

constexpr int kRowT = 256;  // lanes per workgroup
constexpr int kRows = 4;    // rows per workgroup

struct RowArgs {
  int n;
  const double* x;  // [3][n]
  const double* m;  // [n]
  const double* w;  // [3][n] velocities or cotangent
  const double* u;  // [3][n] accelerations (snap)
  double e2;
};

// The double at a byte offset from a base that is the same for every lane: the
// base stays scalar and one offset serves all of a record's arrays.
__device__ __forceinline__ double at_off(const double* base, unsigned off) {
  return *reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + off);
}

// The evaluations: NC sums per row, NW doubles per record.  w[0 .. 2] is the
// position, w[3] the mass, then velocity or cotangent and acceleration; row() and
// rec() load them, past() is a record past the end: far away and massless, so
// its terms are exact zeros.
template <int NW>
struct RowRec {
  double w[NW];
  static __device__ __forceinline__ RowRec at(const RowArgs& A, unsigned off) {
    RowRec r;
#pragma unroll
    for (int c = 0; c < 3; ++c) r.w[c] = at_off(A.x + (size_t)c * A.n, off);
    r.w[3] = at_off(A.m, off);
#pragma unroll
    for (int c = 4; c < NW; ++c) r.w[c] = at_off(c < 7 ? A.w + (size_t)(c - 4) * A.n : A.u + (size_t)(c - 7) * A.n, off);
    return r;
  }
  static __device__ __forceinline__ RowRec past() {
    RowRec r;
#pragma unroll
    for (int c = 0; c < NW; ++c) r.w[c] = c < 3 ? 1.0e30 : 0.0;
    return r;
  }
};

struct RowAccel {
  static constexpr int NC = 3, NW = 4;
  static __device__ __forceinline__ void pair(const RowRec<NW>& r, const RowRec<NW>& s, double e2, bool self, double* p) {
    const double dx = r.w[0] - s.w[0], dy = r.w[1] - s.w[1], dz = r.w[2] - s.w[2];
    double f = r.w[3] * rsqrt64_cubed(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
    f = self ? 0.0 : f;
    p[0] = fma(f, dx, p[0]);
    p[1] = fma(f, dy, p[1]);
    p[2] = fma(f, dz, p[2]);
  }
};

struct RowJerk {
  static constexpr int NC = 6, NW = 7;
  static __device__ __forceinline__ void pair(const RowRec<NW>& r, const RowRec<NW>& s, double e2, bool self, double* p) {
    jerk_pair<double>(r.w[0] - s.w[0], r.w[1] - s.w[1], r.w[2] - s.w[2], r.w[4] - s.w[4], r.w[5] - s.w[5],
                      r.w[6] - s.w[6], r.w[3], e2, self, p, p + 3);
  }
};

struct RowSnap {
  static constexpr int NC = 9, NW = 10;
  static __device__ __forceinline__ void pair(const RowRec<NW>& r, const RowRec<NW>& s, double e2, bool self, double* p) {
    const double d[3] = {r.w[0] - s.w[0], r.w[1] - s.w[1], r.w[2] - s.w[2]};
    const double w[3] = {r.w[4] - s.w[4], r.w[5] - s.w[5], r.w[6] - s.w[6]};
    const double u[3] = {r.w[7] - s.w[7], r.w[8] - s.w[8], r.w[9] - s.w[9]};
    snap_pair<double>(d, w, u, r.w[3], e2, self, p, p + 3, p + 6);
  }
};

struct RowVjp {
  static constexpr int NC = 4, NW = 7;
  static __device__ __forceinline__ void pair(const RowRec<NW>& r, const RowRec<NW>& s, double e2, bool self, double* p) {
    vjp_pair<double>(r.w[0] - s.w[0], r.w[1] - s.w[1], r.w[2] - s.w[2], e2, r.w[3], r.w[4], r.w[5], r.w[6], s.w[3],
                     s.w[4], s.w[5], s.w[6], self, p[0], p[1], p[2], p[3]);
  }
};

// The potential sum m_j s^-1/2; its callers always leave the own pair out.
struct RowPot {
  static constexpr int NC = 1, NW = 4;
  static __device__ __forceinline__ void pair(const RowRec<NW>& r, const RowRec<NW>& s, double e2, bool self, double* p) {
    const double dx = r.w[0] - s.w[0], dy = r.w[1] - s.w[1], dz = r.w[2] - s.w[2];
    const double v = r.w[3] * rsqrt64(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
    p[0] += self ? 0.0 : v;
  }
};

// Grid: ceil(n / kRows) workgroups of kRowT lanes; U records per lane are loaded
// before any is used.
template <class E, int U, bool EXCL, class Epi>
__global__ __launch_bounds__(kRowT) void rows64_kernel(RowArgs A, Epi epi) {
  constexpr int NC = E::NC, M = kRows * NC;
  using Rec = RowRec<E::NW>;
  __shared__ double s_part[M][64];
  __shared__ double s_tot[M];
  const int t = threadIdx.x;
  const int i0 = blockIdx.x * kRows;
  Rec s[kRows];
#pragma unroll
  for (int k = 0; k < kRows; ++k) s[k] = Rec::at(A, 8u * (unsigned)min(i0 + k, A.n - 1));
  double p[M];
#pragma unroll
  for (int q = 0; q < M; ++q) p[q] = 0.0;
  for (int jb = 0; jb < A.n; jb += U * kRowT) {
    Rec r[U];
    if (jb + U * kRowT <= A.n) {  // the same for every lane: no tests in whole blocks
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = Rec::at(A, 8u * (unsigned)(jb + u * kRowT + t));
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        r[u] = Rec::past();
        if (jb + u * kRowT + t < A.n) r[u] = Rec::at(A, 8u * (unsigned)(jb + u * kRowT + t));
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int j = jb + u * kRowT + t;
      if (jb + u * kRowT >= A.n) break;  // the same for every lane
#pragma unroll
      for (int k = 0; k < kRows; ++k) E::pair(r[u], s[k], A.e2, EXCL && j == i0 + k, p + k * NC);
    }
  }
  block_sums<M>(p, s_part, s_tot);
  __syncthreads();
  constexpr int kOuts = Epi::template outs<NC>();
  if (t < kRows * kOuts) {
    const int k = t % kRows, c = t / kRows;
    if (i0 + k < A.n) epi.template apply<NC>(A.n, i0 + k, c, s_tot + k * NC);
  }
}

}  // namespace
}  // namespace nb
