// Row evaluations of small FP32C and FP32 systems: the device side (rows32.hip
// launches it).
//
// As in rows64.h a workgroup evaluates its rows against every j in one launch,
// finishes their sums and does what follows them, but the terms are summed in
// the order of the tile kernels (pairs.hip): one lane adds the 64 terms of a block
// of j one after another in FP32, with the near-field repair of that block, and
// blocks are combined in higher precision.  So the unit of work is a row and a
// block of 64 j, and a wave takes kI rows and 64 / kI blocks at a time: its lanes
// are 64 / kI groups of kI rows, each group with its own block in LDS (staged by
// the wave itself, so the loop has no barrier; a group's records start one
// 16-byte unit further on, so that the groups' reads fall into different banks).
// The groups' sums are added in FP64 by exchanging halves of the wave, the waves'
// in order.
//
// The tile kernel put a block's rescan (the near-field repair, entered by the
// block of the lane's own pair) on the one lane's chain that the launch waits for,
// and the slice sums, the flags of the FP64 rescue and the rescue itself each had
// a launch of their own.  Here the own pair is left out of its block's minimum, so
// only real close pairs rescan; a workgroup flags its own rows and recomputes them
// with all its lanes before it stores them.
//
// Bound: up to ~2000 particles the latency of one launch and one lane's chain of 64
// terms (about 5.5 cycles an instruction with one wave per SIMD), above that VALU
// issue, with 16 waves per workgroup and two workgroups per CU where two fit into its
// 160 KB of LDS: the force (66 KB) and the FP32 jerk and VJP; FP32C jerk and VJP (97 KB)
// and the snap (97 and 129 KB) have one.  FP32C in us, tile
// kernels with their slice sums, flags and rescue -> rows: force 27.9 -> 9.9 at
// 1000, 37 -> 16 at 4096, 80 -> 35 at 8191, 195 -> 87 at 14336; jerk 28 -> 11.4 at
// 1000, 34 -> 24 at 4096, 78 -> 67 at 8191; VJP 30 -> 12.7, 36 -> 26, 85 -> 75; snap
// 41 -> 17, 53 -> 34, 131 -> 110.  The tile kernel's time hung on how evenly its
// j-slices filled the CUs (14336 particles took longer than 16384).
#pragma once

#include "pair_math.h"
#include "row_update.h"
#include "wave64.h"

namespace nb {
namespace {

constexpr int kJBlock = kFold;  // j per block

struct Row32Args {
  int n;
  const double* x;  // [3][n]
  const double* m;  // [n]
  const double* w;  // [3][n] velocities or cotangent
  const double* u;  // [3][n] accelerations (snap)
  double eps, G;    // G: for the flags of the rescue
};

// A row's values: rounded position and its lo part, and what its evaluation needs
// besides (own mass, velocity or cotangent, acceleration).
struct Row32 {
  float h[3], l[3], m, w[3], u[3];
  float rc2, xinf;
};

// The evaluations: NC sums per row, NR float4 arrays of records (position and mass;
// velocity or cotangent; acceleration).  pair() adds the term of displacement d and
// returns the softened squared distance.
struct Row32Accel {
  static constexpr int NC = 3, NR = 1;
  static constexpr bool kChoose = false;
  static __device__ __forceinline__ float pair(const float* d, const float4* r, const Row32&, float e2, bool self, float* p) {
    const float r2 = fma(d[2], d[2], fma(d[1], d[1], fma(d[0], d[0], e2)));
    const float ri = rsq(r2);
    float s = (r[0].w * ri) * (ri * ri);
    if (self) s = 0.f;
    p[0] = fma(s, d[0], p[0]);
    p[1] = fma(s, d[1], p[1]);
    p[2] = fma(s, d[2], p[2]);
    return r2;
  }
};

struct Row32Jerk {
  static constexpr int NC = 6, NR = 2;
  static constexpr bool kChoose = true;
  static __device__ __forceinline__ float pair(const float* d, const float4* r, const Row32& s, float e2, bool self, float* p) {
    return jerk_pair<float>(d[0], d[1], d[2], r[1].x - s.w[0], r[1].y - s.w[1], r[1].z - s.w[2], r[0].w, e2, self, p, p + 3);
  }
};

struct Row32Snap {
  static constexpr int NC = 9, NR = 3;
  static constexpr bool kChoose = true;
  static __device__ __forceinline__ float pair(const float* d, const float4* r, const Row32& s, float e2, bool self, float* p) {
    const float w[3] = {r[1].x - s.w[0], r[1].y - s.w[1], r[1].z - s.w[2]};
    const float u[3] = {r[2].x - s.u[0], r[2].y - s.u[1], r[2].z - s.u[2]};
    return snap_pair<float>(d, w, u, r[0].w, e2, self, p, p + 3, p + 6);
  }
};

struct Row32Vjp {
  static constexpr int NC = 4, NR = 2;
  static constexpr bool kChoose = true;
  static __device__ __forceinline__ float pair(const float* d, const float4* r, const Row32& s, float e2, bool self, float* p) {
    return vjp_pair<float>(d[0], d[1], d[2], e2, r[0].w, r[1].x, r[1].y, r[1].z, s.m, s.w[0], s.w[1], s.w[2], self, p[0],
                           p[1], p[2], p[3]);
  }
};

// The sums p (zero on entry) of one row over the block of 64 records rec
// ([NR][64], with NEAR a last array of lo parts), own the row's index within the
// block (or out of 0 .. 63).  OWN: some lane of the wave has its own pair in its
// block.  The smallest squared distance of a pair left in rounded positions goes
// to r2min.
//
// NEAR repairs the close pairs with the tile kernels' arithmetic.  The force
// replaces a close pair's term after the block's sum; the others sum the block with
// the pair's float-float displacement in its place, chosen here pair by pair (about
// ten operations more on 30 to 60, where a second pass over a block doubled it and
// in these systems most waves met a close pair: jerk 17.3 -> 11.4 us at 1000, 34 ->
// 24.5 at 4096).  The force marks its close pairs, in small systems (SMALL) as it
// goes (three operations on 13: 8.8 against 10.3 us at 1000, but 15.3 against 14.7
// at 4096), else in a second pass over a block that holds one, and then corrects
// them one by one: as many turns as the lane with most of them needs, not one for
// every j that is close to some lane.  Where a block took more than kDense turns (far
// from the origin most pairs are close, the radius grows with |x|) the wave's next
// block is corrected in step, in one pass without marks (dense).
constexpr int kDense = 24;
template <class E, bool NEAR, bool SMALL, bool EXCL, bool OWN>
__device__ __forceinline__ void row32_block(const float4* rec, int own, const Row32& s, float e2, float (&p)[E::NC],
                                            float& r2min, bool& dense) {
  const float4* lo = rec + E::NR * kJBlock;
  unsigned close[2] = {0u, 0u};  // pair jj of each half at bit 31 - jj
  auto sq = [&](const float* d) { return fma(d[2], d[2], fma(d[1], d[1], fma(d[0], d[0], e2))); };
  auto load = [&](int jj, float4* r, float* d) {
#pragma unroll
    for (int q = 0; q < E::NR; ++q) r[q] = rec[q * kJBlock + jj];
    d[0] = r[0].x - s.h[0];
    d[1] = r[0].y - s.h[1];
    d[2] = r[0].z - s.h[2];
  };
  auto full = [&](int jj, const float* d, float* e) {
    const float4 l = lo[jj];
    e[0] = d[0] + (l.x - s.l[0]);
    e[1] = d[1] + (l.y - s.l[1]);
    e[2] = d[2] + (l.z - s.l[2]);
  };
  auto is_self = [&](int jj) { return EXCL && OWN && jj == own; };
  // the pair's term with the displacement that its rounded distance asks for
  auto chosen = [&](int jj) {
    float4 r[E::NR];
    float d[3], e[3];
    load(jj, r, d);
    full(jj, d, e);
    const bool near = sq(d) < s.rc2;
#pragma unroll
    for (int c = 0; c < 3; ++c) d[c] = near ? e[c] : d[c];
    E::pair(d, r, s, e2, is_self(jj), p);
  };
  auto mark = [&](int jj, float r2) {
    const bool near = r2 < s.rc2;
    close[jj / 32] = 2u * close[jj / 32] + (near && !(OWN && jj == own) ? 1u : 0u);
    r2min = fminf(r2min, near ? 3.0e38f : r2);
  };
  r2min = 3.0e38f;
  if constexpr (NEAR && E::kChoose) {
#pragma unroll 8
    for (int jj = 0; jj < kJBlock; ++jj) chosen(jj);
    return;
  }
#pragma unroll 16
  for (int jj = 0; jj < kJBlock; ++jj) {
    float4 r[E::NR];
    float d[3];
    load(jj, r, d);
    const float r2 = E::pair(d, r, s, e2, is_self(jj), p);
    if constexpr (NEAR && SMALL) mark(jj, r2);
    else if constexpr (NEAR) r2min = fminf(r2min, OWN && jj == own ? 3.0e38f : r2);
  }
  if constexpr (NEAR) {
    // p with the rounded term of displacement d replaced by that of the full one
    auto correct = [&](int jj, const float4* r, const float* d, bool near) {
      float e[3];
      full(jj, d, e);
      const float ri = rsq(sq(d)), qi = rsq(sq(e));
      const float f = (r[0].w * ri) * (ri * ri), g = (r[0].w * qi) * (qi * qi);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const float q = fma(g, e[c], fma(-f, d[c], p[c]));
        p[c] = near ? q : p[c];
      }
    };
    if (dense) {
      if (!(r2min < s.rc2)) return;
      r2min = 3.0e38f;
      int many = 0;
#pragma unroll 4
      for (int jj = 0; jj < kJBlock; ++jj) {
        float4 r[E::NR];
        float d[3];
        load(jj, r, d);
        const float r2 = sq(d);
        const bool near = r2 < s.rc2;
        r2min = fminf(r2min, near ? 3.0e38f : r2);
        many += near ? 1 : 0;
        correct(jj, r, d, near && !(OWN && jj == own));
      }
      dense = __any(many > kDense);
      return;
    }
    if (!SMALL && r2min < s.rc2) {
      r2min = 3.0e38f;
#pragma unroll 16
      for (int jj = 0; jj < kJBlock; ++jj) {
        float4 r[E::NR];
        float d[3];
        load(jj, r, d);
        mark(jj, sq(d));
      }
    }
    dense = !SMALL && __any(__popc(close[0]) + __popc(close[1]) > kDense);
#pragma unroll
    for (int half = 0; half < 2; ++half)
      while (close[half]) {
        const int bit = __clz((int)close[half]), jj = half * 32 + bit;
        close[half] &= ~(0x80000000u >> bit);
        float4 r[E::NR];
        float d[3];
        load(jj, r, d);
        correct(jj, r, d, true);
      }
  }
}

// The FP64 sums over all j of the first R of the rows i0 + k, bit k of mask, by the whole
// workgroup (the rescue), into out[k V .. k V + 2]; red holds 3 R doubles per wave.  The
// workgroup's lanes take j in turn, lane sums are added over the wave and the waves in
// order.  Returns the mask without these rows.
template <int R, int V>
__device__ __forceinline__ unsigned row32_rescue(const Row32Args& A, int i0, unsigned mask, bool excl, double* red,
                                                 double* out) {
  const int t = threadIdx.x, T = blockDim.x;
  const double e2 = A.eps * A.eps;
  int row[R];
  double xi[R][3], v[3 * R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    row[k] = mask ? __ffs((int)mask) - 1 : row[k > 0 ? k - 1 : 0];
    mask &= mask - 1;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      xi[k][c] = A.x[(size_t)c * A.n + i0 + row[k]];
      v[3 * k + c] = 0.0;
    }
  }
  for (int j = t; j < A.n; j += T) {
    const double xj = A.x[j], yj = A.x[A.n + j], zj = A.x[2 * (size_t)A.n + j], mj = A.m[j];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const double dx = xj - xi[k][0], dy = yj - xi[k][1], dz = zj - xi[k][2];
      double f = mj * rsqrt64_cubed(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
      if (excl && j == i0 + row[k]) f = 0.0;
      v[3 * k] = fma(f, dx, v[3 * k]);
      v[3 * k + 1] = fma(f, dy, v[3 * k + 1]);
      v[3 * k + 2] = fma(f, dz, v[3 * k + 2]);
    }
  }
  wave_sums<3 * R>(v, red + 3 * R * (t / 64));
  __syncthreads();
  if (t < 3 * R) {
    double s = red[t];
    for (int w = 1; w < T / 64; ++w) s += red[3 * R * w + t];
    int k = row[0];
#pragma unroll
    for (int q = 1; q < R; ++q) k = t / 3 == q ? row[q] : k;
    out[k * V + t % 3] = s;
  }
  __syncthreads();
  return mask;
}

// float4s of a group of I lanes in LDS, and bytes of dynamic LDS of W waves.
template <class E, bool NEAR>
constexpr int row32_group() {
  return (E::NR + (NEAR ? 1 : 0)) * kJBlock + 1;
}
template <class E, int I, bool NEAR>
constexpr size_t row32_lds(int W) {
  return (size_t)W * (64 / I) * row32_group<E, NEAR>() * sizeof(float4);
}

// Grid: ceil(n / I) workgroups of W = blockDim.x / 64 waves.  EST (the FP32C force
// with the rescue): the rows' rounding-error estimates (see rescue.hip), and the
// rows flagged by them in FP64.
template <class E, int I, bool NEAR, bool SMALL, bool EXCL, bool EST, class Epi>
__global__ __launch_bounds__(1024, E::NR == 1 ? 8 : E::NR == 2 ? 7 : 5) void rows32_kernel(Row32Args A, Epi epi) {
  constexpr int GW = 64 / I;                      // groups (blocks of j) per wave
  constexpr int NC = E::NC, V = NC + (EST ? 1 : 0);
  constexpr int kGroup = row32_group<E, NEAR>();
  extern __shared__ float4 s_rec[];
  __shared__ double s_tot[I * V];
  __shared__ unsigned s_mask;
  const int t = threadIdx.x, lane = t & 63, wave = t / 64, W = blockDim.x / 64;
  const int grp = lane / I, li = lane % I;
  const int i0 = blockIdx.x * I, i = i0 + li, n = A.n;
  const float e2 = (float)(A.eps * A.eps);
  float4* const rec = s_rec + (size_t)wave * GW * kGroup;

  Row32 s;
  {
    const int ic = i < n ? i : n - 1;
    double xa[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      xa[c] = A.x[(size_t)c * n + ic];
      s.h[c] = (float)xa[c];
      s.l[c] = (float)(xa[c] - (double)s.h[c]);
      if constexpr (E::NR > 1) s.w[c] = (float)A.w[(size_t)c * n + ic];
      if constexpr (E::NR > 2) s.u[c] = (float)A.u[(size_t)c * n + ic];
    }
    s.m = (float)A.m[ic];
    s.rc2 = near_rc2(xa[0], xa[1], xa[2], A.eps, n);
    s.xinf = (float)fmax(fabs(xa[0]), fmax(fabs(xa[1]), fabs(xa[2])));
  }
  float hi[NC], lo[NC], eacc = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) hi[c] = lo[c] = 0.f;

  const int nblk = (n + kJBlock - 1) / kJBlock, ownb = i0 / kJBlock;
  bool dense = false;
  for (int b0 = wave * GW; b0 < nblk; b0 += W * GW) {
    // the wave's GW blocks of records, padding past n far away and massless
    wave_sync();
#pragma unroll
    for (int q = 0; q < GW; ++q) {
      const int j = (b0 + q) * kJBlock + lane;
      const bool in = j < n;
      const int jc = in ? j : n - 1;
      float4 r[E::NR + 1];
      const double xj = in ? A.x[jc] : kFarAway, yj = in ? A.x[n + jc] : kFarAway,
                   zj = in ? A.x[2 * (size_t)n + jc] : kFarAway;
      r[0] = make_float4((float)xj, (float)yj, (float)zj, in ? (float)A.m[jc] : 0.f);
      r[E::NR] = make_float4((float)(xj - (double)r[0].x), (float)(yj - (double)r[0].y), (float)(zj - (double)r[0].z), 0.f);
      if constexpr (E::NR > 1)
        r[1] = in ? make_float4((float)A.w[jc], (float)A.w[n + jc], (float)A.w[2 * (size_t)n + jc], 0.f)
                  : make_float4(0.f, 0.f, 0.f, 0.f);
      if constexpr (E::NR > 2)
        r[2] = in ? make_float4((float)A.u[jc], (float)A.u[n + jc], (float)A.u[2 * (size_t)n + jc], 0.f)
                  : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < E::NR + (NEAR ? 1 : 0); ++k) rec[q * kGroup + k * kJBlock + lane] = r[k];
    }
    wave_sync();
    float p[NC], r2min;
#pragma unroll
    for (int c = 0; c < NC; ++c) p[c] = 0.f;
    // the workgroup's rows lie in one block of j: its wave leaves the own pairs out
    if (ownb >= b0 && ownb < b0 + GW) row32_block<E, NEAR, SMALL, EXCL, true>(rec + grp * kGroup, i - (b0 + grp) * kJBlock, s, e2, p, r2min, dense);
    else row32_block<E, NEAR, SMALL, EXCL, false>(rec + grp * kGroup, -1, s, e2, p, r2min, dense);
    if constexpr (EST) eacc = est_add(eacc, p[0], p[1], p[2], s.xinf, r2min);
#pragma unroll
    for (int c = 0; c < NC; ++c) fold(hi[c], lo[c], p[c]);
  }

  // the wave's groups in FP64, then the waves in order
  double v[V];
#pragma unroll
  for (int c = 0; c < NC; ++c) v[c] = (double)hi[c] + (double)lo[c];
  if constexpr (EST) v[NC] = (double)eacc;
  constexpr int kWave = GW * kGroup * 2;  // doubles between the waves' sums, which take their records' place
  static_assert(kWave >= V * I, "a wave's sums fit where its records were");
  double* const red = reinterpret_cast<double*>(s_rec);
  wave_sync();
  group_sums<I, V>(v, red + (size_t)wave * kWave);
  __syncthreads();
  for (int q = t; q < V * I; q += blockDim.x) {
    double a = red[q];
    for (int w = 1; w < W; ++w) a += red[(size_t)w * kWave + q];
    s_tot[(q % I) * V + q / I] = a;
  }
  __syncthreads();
  if constexpr (EST) {
    if (t < 64) {
      bool flag = false;
      if (t < I && i0 + t < n) {
        const double* a = s_tot + t * V;
        const double ax = A.G * a[0], ay = A.G * a[1], az = A.G * a[2];
        flag = sqrt(a[3]) * (kRescueScale * fabs(A.G)) > sqrt(ax * ax + ay * ay + az * az);
      }
      const unsigned long long mask = __ballot(flag);
      if (t == 0) s_mask = (unsigned)mask;
    }
    __syncthreads();
    // two rows on each record read (four at a time spill scalar registers, which costs the
    // smallest systems up to 8 %)
    for (unsigned mask = (unsigned)__builtin_amdgcn_readfirstlane((int)s_mask); mask;)
      mask = mask & (mask - 1) ? row32_rescue<2, V>(A, i0, mask, EXCL, red, s_tot)
                               : row32_rescue<1, V>(A, i0, mask, EXCL, red, s_tot);
  }
  constexpr int kOuts = Epi::template outs<NC>();
  for (int q = t; q < I * kOuts; q += blockDim.x) {
    const int k = q % I;
    if (i0 + k < n) epi.template apply<NC>(n, i0 + k, q / I, s_tot + k * V);
  }
}

}  // namespace
}  // namespace nb
