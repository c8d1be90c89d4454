// Rescue of ill-conditioned rows of the FP32C force.
//
// An FP32C row a_i is a sum of FP32 pair terms, each carrying a relative
// rounding error of a few u (u = 2^-24): the inverse square root, its cube,
// the weight and the products, and, for pairs outside the near-field radius,
// the rounding of both positions to FP32, which moves the displacement by up
// to about u (|x_i| + |x_j|).  Where the terms of a row cancel (|a_i| much
// smaller than the sum of their magnitudes, e.g. particles near the centre of
// a cluster) those errors are large relative to |a_i|; the largest come from
// strong pairs just outside the near-field radius, whose terms keep the
// rounding of both positions.  The pair kernels keep a cheap estimate of each
// row's error: for every block of terms they sum in FP32 (64 terms of the
// row's own j-loop, or, for the far side of the symmetric kernels, one slot of
// up to 512 terms) they add the square of the block's partial sum |P_b|,
// weighted by 1 + kEstNear |x_i|_inf / d_b, d_b the smallest softened distance
// of a pair of that block that was not repaired with float-float
// displacements (for a far-side slot, a lower bound of it: the smallest such
// distance among all pairs of the tile of 64 j the slot belongs to):
//   E_i = sum_b ((1 + kEstNear |x_i| / d_b) |P_b|)^2 .
// The rounding error of a block's sum grows like the magnitude of its partial
// sum both when one term dominates the block and when its terms have random
// directions (both the sum and the error then grow like the square root of the
// number of terms), the distance factor prices the position rounding of the
// block's closest pair, and the errors of different blocks (different j,
// different roundings) add like independent variables, hence the root of the
// sum of squares.  A row is recomputed in FP64 when
//   kEstC u |G| sqrt(E_i) > kRescueTol |a_i| .
// kEstC and kRescueTol were set against measured errors: over half a million
// rows of Plummer spheres (512 to 2^20 particles, softenings down to
// 6.25e-4) and the two-component model, the estimate exceeded the actual
// error of FP32C (without rescue, against FP64) by 4 to 10 at the median and
// the row left unflagged with the largest error stayed at 2.7e-6, against 4e-5
// for the largest error without rescue.  With the far side's per-tile bound,
// 610 000 rows of Plummer spheres (4096 to 262144 particles, softenings
// 6.25e-4 to 1e-3, symmetric kernel) left 2.3e-6 as the largest unflagged
// error with 0.86 % of the rows recomputed; 0.12 % of the rows of the 2^20
// two-component model are.  The estimate misses cancellation that is
// systematic inside one block of consecutive indices (terms of a block that
// cancel each other more than random directions do).
//
// Here, for the force of one system: the flagged rows go to a list (an atomic
// counter, one add per wave, orders them, which does not change any result:
// every row is recomputed on its own, in an order that depends only on how many
// there are) and a grid-stride kernel recomputes them in FP64.  The count of flagged rows is cleared by the
// first kernel of the evaluation (its block 0, thread 0), so that the flag
// kernel starts from zero without a launch of its own.  The batched wave items
// (ensemble_stream.hip) flag their rows in the force kernel, where each wave
// holds whole rows, into per-system lists that their own rescue kernel reads.
#include "pair_math.h"
#include "wave64.h"

namespace nb {
namespace {

// One thread per particle: sums the nslices slices of the estimate (stride
// apart) and appends the row to the list if scale * sqrt(E_i) > |a_i|.  A
// wave reserves the places of all its flagged rows with one atomic add.  The first
// nclear words of the estimate, once read, become the rescue's zeroed arrival counts
// (word i is read by this thread alone).
__global__ void flag_rows_kernel(int n, float* est, int nslices, size_t stride, const double* __restrict__ a,
                                 double scale, int* __restrict__ list, int* __restrict__ count, int nclear) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  bool flag = false;
  if (i < n) {
    float e = 0.f;
    for (int k = 0; k < nslices; ++k) e += est[(size_t)k * stride + i];
    if (i < nclear) est[i] = 0.f;
    const double ax = a[i], ay = a[n + i], az = a[2 * n + i];
    const double an = sqrt(ax * ax + ay * ay + az * az);
    flag = sqrt((double)e) * scale > an;
  }
  const unsigned long long mask = __ballot(flag);
  if (mask == 0) return;
  const int lane = threadIdx.x & 63;
  int base = 0;
  if (lane == __ffsll((long long)mask) - 1) base = atomicAdd(count, __popcll(mask));
  base = __shfl(base, __ffsll((long long)mask) - 1, 64);
  if (flag) list[base + __popcll(mask & ((1ull << lane) - 1ull))] = i;
}

// Recomputes the listed rows of a = G sum_j m_j d / (|d|^2 + eps^2)^(3/2) in
// FP64.  A unit is a group of R listed rows (each j record serves them all) and one
// of S equal runs of j: with few rows S is what fills the chip, up to runs of one
// pass of a workgroup (B U records) and ucap units; with many it is 1.  Units of the
// same run are neighbours, so the workgroups at work at one time read the same
// records out of L2.  The B lanes split a unit's j (lane t takes t, t + B, ...),
// loading U records ahead of the arithmetic, and the lane sums are added in a fixed
// order: inside each wave in registers, then the wave sums in wave order.  With S > 1
// the unit's sums go to part, and the workgroup whose arrival completes the group
// (arrived counts them; no workgroup waits) adds the runs in a fixed order.
//
// Bound by FP64 issue where there are rows enough (21 issue slots a pair), by the
// latency of the loads where there are few.  Against a group of rows per workgroup
// over all j: 38 -> 15 us for the 21 rows of a Plummer sphere of 65536, 1.59 -> 1.27
// ms for the 1367 of the two-component model of 2^20 (1.41 with groups of four).
template <int R, int B, int U>
__global__ __launch_bounds__(B) void rescue_rows_kernel(int n, const double* __restrict__ x,
                                                        const double* __restrict__ m, double eps, double G,
                                                        int excl, const int* __restrict__ list,
                                                        const int* __restrict__ count, double* __restrict__ a,
                                                        int* arrived, double* part, int ucap) {
  constexpr int W = B / 64;
  __shared__ double red[W][R * 3];
  __shared__ int last;
  const int t = threadIdx.x;
  const int wave = t / 64, lane = t % 64;
  const int cnt = *count;
  if (cnt == 0) return;
  const double e2 = eps * eps;
  const int groups = (cnt + R - 1) / R;
  const int S = max(1, min(ucap / groups, (n + B * U - 1) / (B * U)));
  const int len = ((n + S - 1) / S + 63) / 64 * 64;
  for (int unit = blockIdx.x; unit < groups * S; unit += gridDim.x) {
    const int grp = unit % groups, r0 = grp * R;
    const int jbeg = unit / groups * len, jend = min(n, jbeg + len);
    int row[R];
    double xi[R], yi[R], zi[R], sum[3 * R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      row[k] = r0 + k < cnt ? list[r0 + k] : -1;
      const int i = row[k] < 0 ? 0 : row[k];
      xi[k] = x[i];
      yi[k] = x[n + i];
      zi[k] = x[2 * n + i];
      sum[3 * k] = sum[3 * k + 1] = sum[3 * k + 2] = 0.0;
    }
    for (int j0 = jbeg + t; j0 < jend; j0 += U * B) {
      // U records per lane, all loaded before any is used; past the run: far away
      // and massless, so they add exact zeros
      double xj[U], yj[U], zj[U], mj[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * B;
        const bool in = j < jend;
        xj[u] = in ? x[j] : 1.0e30;
        yj[u] = in ? x[n + j] : 1.0e30;
        zj[u] = in ? x[2 * n + j] : 1.0e30;
        mj[u] = in ? m[j] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int j = j0 + u * B;
#pragma unroll
        for (int k = 0; k < R; ++k) {
          const double dx = xj[u] - xi[k], dy = yj[u] - yi[k], dz = zj[u] - zi[k];
          const double r2 = fma(dz, dz, fma(dy, dy, fma(dx, dx, e2)));
          const double ri = rsqrt64(r2);
          double s = (mj[u] * ri) * (ri * ri);
          if (excl && j == row[k]) s = 0.0;
          sum[3 * k] = fma(s, dx, sum[3 * k]);
          sum[3 * k + 1] = fma(s, dy, sum[3 * k + 1]);
          sum[3 * k + 2] = fma(s, dz, sum[3 * k + 2]);
        }
      }
    }
    wave_sums(sum, red[wave]);
    __syncthreads();
    // lane t < 3 R: row t / 3, component t % 3
    double v = 0.0;
    if (t < 3 * R) {
      v = red[0][t];
#pragma unroll
      for (int w = 1; w < W; ++w) v += red[w][t];
      if (S > 1)
        __hip_atomic_store(&part[(size_t)unit * 3 * R + t], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (S > 1) {
      __syncthreads();
      if (t == 0)
        last = __hip_atomic_fetch_add(&arrived[grp], 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == S - 1;
      __syncthreads();
      if (last) {
        // wave w adds the runs w, w + W, ..., then the waves' sums in wave order
        if (lane < 3 * R) {
          v = 0.0;
          for (int q = wave; q < S; q += W) v += part[((size_t)q * groups + grp) * 3 * R + lane];
          red[wave][lane] = v;
        }
        __syncthreads();
        if (t < 3 * R) {
          v = red[0][t];
#pragma unroll
          for (int w = 1; w < W; ++w) v += red[w][t];
        }
      }
    }
    if (t < 3 * R && r0 + t / 3 < cnt && (S == 1 || last)) a[(size_t)(t % 3) * n + list[r0 + t / 3]] = G * v;
    __syncthreads();
  }
}

// Rows of a group, lanes per workgroup and records loaded ahead.
constexpr int kRRows = 8, kRLanes = 512, kRAhead = 2;
// Units of a rescue with runs of j, at most; their counts and sums lie in the
// estimate's own memory (n floats), which the flagging has read by then.
constexpr int64_t kRUnits = 8192;

}  // namespace

int launch_rescue(int64_t n, const double* x, const double* m, double eps, double G, bool excl, float* est,
                  int nslices, size_t stride, double* a, int* list, int* count, hipStream_t s) {
  if (n == 0) return NBODY_OK;
  const double scale = kRescueScale * std::fabs(G);
  // a group has runs (S > 1) only if there are at most ucap / 2 groups
  constexpr int64_t unit_bytes = 3 * kRRows * (int64_t)sizeof(double);
  const int64_t ucap = n < 1024 ? 0 : std::min<int64_t>(kRUnits, n * (int64_t)sizeof(float) / (unit_bytes + 4));
  const int64_t nclear = ucap / 2;
  double* part = reinterpret_cast<double*>(est + (nclear + 1) / 2 * 2);
  flag_rows_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>((int)n, est, nslices, stride, a, scale, list, count,
                                                               (int)nclear);
  NB_LAUNCH_CHECK("flag_rows_kernel");
  // about as many workgroups as are resident at once; each strides over the units
  const unsigned grid = (unsigned)std::min<int64_t>((n + kRRows - 1) / kRRows + ucap, 2 * (int64_t)cu_count(current_device()));
  rescue_rows_kernel<kRRows, kRLanes, kRAhead><<<grid, kRLanes, 0, s>>>((int)n, x, m, eps, G, excl ? 1 : 0, list, count,
                                                                        a, reinterpret_cast<int*>(est), part,
                                                                        (int)ucap);
  NB_LAUNCH_CHECK("rescue_rows_kernel");
  return NBODY_OK;
}

}  // namespace nb
