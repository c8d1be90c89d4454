// Symmetric FP64 evaluations: every unordered pair once, its terms applied to both
// particles, on the layout of the FP32C kernel (sym_pairs.hip): I-blocks of 512
// particles, two per lane; J-blocks streamed through LDS in tiles of 64 as
// sub-blocks of 16 stored twice in a row, so that at step K lane r meets record
// (r + K) mod 16; the j-side terms of both i of a lane summed and moved to the
// lane owning that j by a row rotation (each double as two 32-bit DPP moves, then
// an FP64 add); tile sums to per-distance FP64 slots; a half ring of block pairs
// in chunks; FP64 slot sums in a fixed order.  All arithmetic is FP64; there is no
// near-field repair to do.
//
// One kernel serves the force (three components per particle), its
// vector-Jacobian product (four), acceleration + jerk (six), acceleration + jerk +
// snap (nine) and the potential (one); an evaluation gives its pair terms.
//
// Bound: FP64 issue.  What keeps the other units out of its way:
//   * a record lies in LDS as pairs of doubles in arrays of their own, so that the
//     16 records a row reads at a step cover the banks once (as records of four
//     doubles the lanes eight apart met in the same banks);
//   * the far-side sums of a sub-block are added over the four rows of a wave by
//     exchanging halves in registers (three operations a value and level, and one
//     LDS write for up to four components) instead of two LDS round trips a value;
//   * the block with itself (distance 0) is a share of the same launch, its
//     workgroups first: as a kernel of its own it held a small ring's launch up by
//     its whole length, and on a second stream by the waits.
// Before (one kernel per evaluation, records of four doubles, LDS reductions, the
// diagonal kernel) -> after, in us: force 82.6 -> 69 at 9973, 100 -> 90 at 12000,
// 1860 -> 1853 at 65536, 29.8 -> 28.0 ms at 262144; VJP 143 -> 114 at 9973, 825 ->
// 790 at 30011, 56.6 -> 55.4 ms at 262144; acceleration + jerk 133 -> 107 and 763 ->
// 726; acceleration + jerk + snap 211 -> 168 and 1320 -> 1265; potential 84.6
// (ordered) -> 50 and 528 -> 272.
#include <mutex>

#include "sym_common.h"
#include "wave64.h"

namespace nb {
namespace {

struct Sym64Args {
  const double2* rec;  // staged records: 2 NR arrays [npad]: (x, y), (z, m), (wx, wy), (wz, 0), (ux, uy), (uz, 0)
  int nb, npad, dmax, half, d_lo, T, nparts;  // T: tiles per workgroup
  int ndiag, Td;       // workgroups of the blocks with themselves (0: none in this launch), tiles of each
  int excl;
  double e2;
  double* pj;          // [D][NC][npad] j-side tile sums of the chunk's distances
  double* pi;          // [nparts][NC][npad] i-side sums of the chunk's workgroups
  double* pd;          // [kSTiles / Td][NC][npad] sums of the blocks with themselves
};

// The evaluations: NC components, NR records of four doubles, the waves per SIMD
// the kernel is built for.  pair() takes record r and particle s (as staged), adds
// i's terms to p and j's to t; own leaves the own pair out, whose factors are then
// zeros (without softening they are infinite or NaN).  kOwn: the own pair is always
// left out, not only where asked (with softening the others' own terms are zero).

// a_i += m_j r^-3 d, a_j -= m_i r^-3 d, d = x_j - x_i, r^2 = |d|^2 + eps^2.
struct Sym64Accel {
  static constexpr int NC = 3, NR = 1, kWaves = 5;
  static constexpr bool kOwn = false;
  static __device__ __forceinline__ void pair(const double* r, const double* s, double e2, bool own, double* p, double* t) {
    const double dx = r[0] - s[0], dy = r[1] - s[1], dz = r[2] - s[2];
    double f = rsqrt64_cubed(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
    f = own ? 0.0 : f;
    const double si = r[3] * f, sj = -s[3] * f;
    p[0] = fma(si, dx, p[0]);
    p[1] = fma(si, dy, p[1]);
    p[2] = fma(si, dz, p[2]);
    t[0] = fma(sj, dx, t[0]);
    t[1] = fma(sj, dy, t[1]);
    t[2] = fma(sj, dz, t[2]);
  }
};

// phi_i += m_j r^-1, phi_j += m_i r^-1: a pair evaluation of 13 FP64 operations and
// one v_rsq_f64 replaces two of 14 and 1.
struct Sym64Pot {
  static constexpr int NC = 1, NR = 1, kWaves = 8;
  static constexpr bool kOwn = true;
  static __device__ __forceinline__ void pair(const double* r, const double* s, double e2, bool own, double* p, double* t) {
    const double dx = r[0] - s[0], dy = r[1] - s[1], dz = r[2] - s[2];
    double ri = rsqrt64(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
    ri = own ? 0.0 : ri;
    p[0] = fma(r[3], ri, p[0]);
    t[0] = fma(s[3], ri, t[0]);
  }
};

// With u = m_k w_j - m_j w_k:
//   gx_k += r^-3 u - 3 r^-5 (d.u) d,   gm_k -= r^-3 (d . w_j),
//   gx_j -= r^-3 u - 3 r^-5 (d.u) d,   gm_j += r^-3 (d . w_k)
// (d and u both change sign when k and j swap).
struct Sym64Vjp {
  static constexpr int NC = 4, NR = 2, kWaves = 4;
  static constexpr bool kOwn = true;
  static __device__ __forceinline__ void pair(const double* r, const double* s, double e2, bool own, double* p, double* t) {
    const double dx = r[0] - s[0], dy = r[1] - s[1], dz = r[2] - s[2];
    const double ri = rsqrt64(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
    const double ri2 = ri * ri;
    const double r3 = own ? 0.0 : ri2 * ri;
    const double c5 = own ? 0.0 : (-3.0 * ri2) * r3;
    const double ux = fma(s[3], r[4], -(r[3] * s[4]));
    const double uy = fma(s[3], r[5], -(r[3] * s[5]));
    const double uz = fma(s[3], r[6], -(r[3] * s[6]));
    const double cc = c5 * fma(dz, uz, fma(dy, uy, dx * ux));
    p[0] = fma(cc, dx, fma(r3, ux, p[0]));
    p[1] = fma(cc, dy, fma(r3, uy, p[1]));
    p[2] = fma(cc, dz, fma(r3, uz, p[2]));
    t[0] = fma(-cc, dx, fma(-r3, ux, t[0]));
    t[1] = fma(-cc, dy, fma(-r3, uy, t[1]));
    t[2] = fma(-cc, dz, fma(-r3, uz, t[2]));
    p[3] = fma(-r3, fma(dz, r[6], fma(dy, r[5], dx * r[4])), p[3]);
    t[3] = fma(r3, fma(dz, s[6], fma(dy, s[5], dx * s[4])), t[3]);
  }
};

// Algorithm 3 with w = v_j - v_i and q = -3 r^-2 (d . w):
//   a_i += m_j r^-3 d,   jerk_i += m_j r^-3 (w + q d),
//   a_j -= m_i r^-3 d,   jerk_j -= m_i r^-3 (w + q d)
// (d and w change sign when i and j swap, q does not).
struct Sym64Jerk {
  static constexpr int NC = 6, NR = 2, kWaves = 2;
  static constexpr bool kOwn = false;
  static __device__ __forceinline__ void pair(const double* r, const double* s, double e2, bool own, double* p, double* t) {
    const double dx = r[0] - s[0], dy = r[1] - s[1], dz = r[2] - s[2];
    const double wx = r[4] - s[4], wy = r[5] - s[5], wz = r[6] - s[6];
    const double ri = rsqrt64(fma(dz, dz, fma(dy, dy, fma(dx, dx, e2))));
    const double ri2 = ri * ri;
    const double r3 = own ? 0.0 : ri2 * ri;
    const double q = own ? 0.0 : (-3.0 * ri2) * fma(dz, wz, fma(dy, wy, dx * wx));
    const double jx = fma(q, dx, wx), jy = fma(q, dy, wy), jz = fma(q, dz, wz);
    const double si = r[3] * r3, sj = -s[3] * r3;
    p[0] = fma(si, dx, p[0]); p[1] = fma(si, dy, p[1]); p[2] = fma(si, dz, p[2]);
    p[3] = fma(si, jx, p[3]); p[4] = fma(si, jy, p[4]); p[5] = fma(si, jz, p[5]);
    t[0] = fma(sj, dx, t[0]); t[1] = fma(sj, dy, t[1]); t[2] = fma(sj, dz, t[2]);
    t[3] = fma(sj, jx, t[3]); t[4] = fma(sj, jy, t[4]); t[5] = fma(sj, jz, t[5]);
  }
};

// The sixth-order Hermite evaluation: with the acceleration difference u and
// alpha = (d . w) / r^2, beta = (w.w + d.u) / r^2 + alpha^2, the per-unit-mass terms
//   p0 = r^-3 d,  p1 = r^-3 w - 3 alpha p0,  p2 = r^-3 u - 6 alpha p1 - 3 beta p0
// (d, w and u change sign when i and j swap, alpha and beta do not).
struct Sym64Snap {
  static constexpr int NC = 9, NR = 3, kWaves = 2;
  static constexpr bool kOwn = false;
  static __device__ __forceinline__ void pair(const double* r, const double* s, double e2, bool own, double* p, double* t) {
    const double d[3] = {r[0] - s[0], r[1] - s[1], r[2] - s[2]};
    const double w[3] = {r[4] - s[4], r[5] - s[5], r[6] - s[6]};
    const double u[3] = {r[8] - s[8], r[9] - s[9], r[10] - s[10]};
    const double ri = rsqrt64(fma(d[2], d[2], fma(d[1], d[1], fma(d[0], d[0], e2))));
    const double sinv = ri * ri;
    const double r3 = own ? 0.0 : sinv * ri;
    const double alpha = own ? 0.0 : fma(d[2], w[2], fma(d[1], w[1], d[0] * w[0])) * sinv;
    const double wwdu = fma(d[2], u[2], fma(d[1], u[1], fma(d[0], u[0], fma(w[2], w[2], fma(w[1], w[1], w[0] * w[0])))));
    const double beta = own ? 0.0 : fma(wwdu, sinv, alpha * alpha);
    const double a3 = -3.0 * alpha, a6 = -6.0 * alpha, b3 = -3.0 * beta;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const double p0 = r3 * d[c];
      const double p1 = fma(a3, p0, r3 * w[c]);
      const double p2 = fma(a6, p1, fma(b3, p0, r3 * u[c]));
      p[c] = fma(r[3], p0, p[c]);
      p[3 + c] = fma(r[3], p1, p[3 + c]);
      p[6 + c] = fma(r[3], p2, p[6 + c]);
      t[c] = fma(-s[3], p0, t[c]);
      t[3 + c] = fma(-s[3], p1, t[3 + c]);
      t[6 + c] = fma(-s[3], p2, t[6 + c]);
    }
  }
};

// A tile's records in LDS: per array of pairs, four sub-blocks of 16, each twice.
template <int NA>
struct Tile64 {
  double2 r[NA][4][2 * kSR];
};

// Step K of sub-block q: both particles of the lane against record (rl + K).  DIAG:
// the lane's block meets itself, i-side only, own0 and own1 telling whether this
// step's pair (K == 0 of the right sub-block) is an own pair.
template <class E, int K, bool DIAG>
__device__ __forceinline__ void sym64_step(const double (&s)[2][4 * E::NR], const Tile64<2 * E::NR>& tile, int q, int rl,
                                           double e2, bool own0, bool own1, double (&p)[2][E::NC], double (&aj)[E::NC]) {
  double r[4 * E::NR];
#pragma unroll
  for (int a = 0; a < 2 * E::NR; ++a) {
    const double2 v = tile.r[a][q][rl + K];
    r[2 * a] = v.x;
    r[2 * a + 1] = v.y;
  }
  double t[E::NC];
#pragma unroll
  for (int c = 0; c < E::NC; ++c) t[c] = 0.0;
  E::pair(r, s[0], e2, DIAG && K == 0 && own0, p[0], t);
  E::pair(r, s[1], e2, DIAG && K == 0 && own1, p[1], t);
  if constexpr (!DIAG) {
    // the j met here sits at row position (rl + K): its owner is K lanes further on
#pragma unroll
    for (int c = 0; c < E::NC; ++c)
      if constexpr (K == 0) aj[c] += t[c];
      else aj[c] += row_ror64<K>(t[c]);
  }
}

template <class E, bool DIAG, int... K>
__device__ __forceinline__ void sym64_sub(const double (&s)[2][4 * E::NR], const Tile64<2 * E::NR>& tile, int q, int rl,
                                          double e2, bool own0, bool own1, double (&p)[2][E::NC], double (&aj)[E::NC],
                                          std::integer_sequence<int, K...>) {
  (sym64_step<E, K, DIAG>(s, tile, q, rl, e2, own0, own1, p, aj), ...);
}

// The records of all npad particles (padding past n: far away, massless, at rest).
template <class E>
__global__ void sym64_stage_kernel(int n, int npad, const double* __restrict__ x, const double* __restrict__ m,
                                   const double* __restrict__ w, const double* __restrict__ u, double2* __restrict__ rec) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= npad) return;
  const bool in = j < n;
  rec[j] = in ? make_double2(x[j], x[(size_t)n + j]) : make_double2(kFarAway, kFarAway);
  rec[(size_t)npad + j] = in ? make_double2(x[2 * (size_t)n + j], m[j]) : make_double2(kFarAway, 0.0);
  if constexpr (E::NR > 1) {
    rec[2 * (size_t)npad + j] = in ? make_double2(w[j], w[(size_t)n + j]) : make_double2(0.0, 0.0);
    rec[3 * (size_t)npad + j] = make_double2(in ? w[2 * (size_t)n + j] : 0.0, 0.0);
  }
  if constexpr (E::NR > 2) {
    rec[4 * (size_t)npad + j] = in ? make_double2(u[j], u[(size_t)n + j]) : make_double2(0.0, 0.0);
    rec[5 * (size_t)npad + j] = make_double2(in ? u[2 * (size_t)n + j] : 0.0, 0.0);
  }
}

template <class E>
struct Sym64Shared {
  Tile64<2 * E::NR> tile[2];
  double part[E::NC][kSW][kST];
  double lo[2 * E::NC][kSL];  // the lo halves of the i-side (hi, lo) sums
};

// Tiles kbeg .. kend - 1 of I-block g: the chunk's ring tiles counted from the first
// tile of distance d_lo, or with DIAG the tiles of block g itself; the i-side sums
// of its particles into out[NC][npad].
template <class E, bool DIAG>
__device__ __forceinline__ void sym64_tiles(const Sym64Args& A, Sym64Shared<E>& sh, int g, int kbeg, int kend, double* out) {
  constexpr int NC = E::NC, NA = 2 * E::NR;
  const int t = threadIdx.x, lane = t & 63, wave = t / 64;
  const int rl = lane & (kSR - 1), row = lane >> 4;

  double s[2][4 * E::NR];
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const double2 q = A.rec[(size_t)a * A.npad + (size_t)g * kSI + v * kSL + t];
      s[v][2 * a] = q.x;
      s[v][2 * a + 1] = q.y;
    }
  double hi[2][NC];
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      hi[v][c] = 0.0;
      sh.lo[v * NC + c][t] = 0.0;
    }

  auto block_of = [&](int k) { return DIAG ? g : (g + A.d_lo + k / kSTiles) % A.nb; };
  // the last wave copies tile k into LDS buffer b straight from global memory, two
  // copies of 64 lanes x 16 bytes per array, which lay two sub-blocks out twice in
  // a row each; the lane's offset enters each address afresh (an empty asm
  // statement hides it from hoisting), so that every copy takes the form scalar
  // base + 32-bit lane offset
  const unsigned lane_off = (unsigned)(((lane >> 5) * kSR + rl) * sizeof(double2));
  auto stage = [&](int k, int b) {
    const int rec0 = __builtin_amdgcn_readfirstlane(block_of(k) * kSI + (k % kSTiles) * kST);
    unsigned o = lane_off;
    asm volatile("" : "+v"(o));
#pragma unroll
    for (int a = 0; a < NA; ++a) {
      const char* base = reinterpret_cast<const char*>(A.rec + (size_t)a * A.npad + rec0);
      __builtin_amdgcn_global_load_lds(base + o, (lds_ptr)&sh.tile[b].r[a][0][0], 16, 0, 0);
      __builtin_amdgcn_global_load_lds(base + 2 * kSR * sizeof(double2) + o, (lds_ptr)&sh.tile[b].r[a][2][0], 16, 0, 0);
    }
  };
  if (kbeg < kend && wave == kSW - 1) {
    stage(kbeg, 0);
    __builtin_amdgcn_s_waitcnt(0);
  }
  __syncthreads();

  for (int k = kbeg; k < kend; ++k) {
    const int b = (k - kbeg) & 1;
    if (wave == kSW - 1 && k + 1 < kend) stage(k + 1, b ^ 1);
    double p[2][NC];
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int c = 0; c < NC; ++c) p[v][c] = 0.0;
#pragma unroll 1
    for (int q = 0; q < 4; ++q) {
      double aj[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) aj[c] = 0.0;
      // particle v of the lane is j = 64 (4 v + wave) + lane of its block, met at
      // step 0 of the sub-block of its own row
      const bool mine = DIAG && q == row && (E::kOwn || A.excl);
      sym64_sub<E, DIAG>(s, sh.tile[b], q, rl, A.e2, mine && k == wave, mine && k == kSW + wave, p, aj,
                         std::make_integer_sequence<int, kSR>{});
      if constexpr (!DIAG) {
        // the four rows' sums of the same 16 j: each group of four components ends
        // up with one in each row (the last repeated where there are fewer, so that
        // every lane stores and nothing branches)
#pragma unroll
        for (int c = 0; c < NC; c += 4) {
          auto at = [&](int i) { return aj[c + i < NC ? c + i : NC - 1]; };
          const double v = swap_add<16>(swap_add<32>(at(0), at(1)), swap_add<32>(at(2), at(3)));
          const int cc = c + 2 * (row & 1) + (row >> 1);
          sh.part[cc < NC ? cc : NC - 1][wave][q * kSR + rl] = v;
        }
      }
    }
#pragma unroll
    for (int v = 0; v < 2; ++v)
#pragma unroll
      for (int c = 0; c < NC; ++c) fold(hi[v][c], sh.lo[v * NC + c][t], p[v][c]);
    __syncthreads();
    if constexpr (!DIAG) {
      // the tile's j-side sums: the four waves' of each j and component, in order
      double* dst = A.pj + (size_t)(k / kSTiles) * NC * A.npad + (size_t)block_of(k) * kSI + (k % kSTiles) * kST;
#pragma unroll
      for (int e = 0; e < NC * kST; e += kSL) {
        const int f = e + t, c = f / kST, jl = f % kST;
        if (NC * kST - e >= kSL || f < NC * kST) {
          double v = 0.0;
#pragma unroll
          for (int w = 0; w < kSW; ++w) v += sh.part[c][w][jl];
          dst[(size_t)c * A.npad + jl] = v;
        }
      }
    }
    if (wave == kSW - 1) __builtin_amdgcn_s_waitcnt(0);  // the next tile's copies have landed in LDS
    __syncthreads();
  }

#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int c = 0; c < NC; ++c)
      out[(size_t)c * A.npad + (size_t)g * kSI + v * kSL + t] = hi[v][c] + sh.lo[v * NC + c][t];
}

// Grid: ndiag + nb * nparts workgroups: those of the blocks with themselves, slice
// by slice, then (g, part) with tiles [part T, (part + 1) T) of I-block g's ring.
template <class E>
__global__ __launch_bounds__(kSL, E::kWaves) void sym64_kernel(Sym64Args A) {
  __shared__ Sym64Shared<E> sh;
  if ((int)blockIdx.x < A.ndiag) {
    const int g = blockIdx.x % A.nb, slice = blockIdx.x / A.nb;
    sym64_tiles<E, true>(A, sh, g, slice * A.Td, (slice + 1) * A.Td, A.pd + (size_t)slice * E::NC * A.npad);
    return;
  }
  const int lid = xcd_local_index((int)blockIdx.x - A.ndiag, (int)gridDim.x - A.ndiag);
  const int g = lid % A.nb, part = lid / A.nb;
  const int rend = (A.half && g >= A.nb / 2) ? A.dmax : A.dmax + 1;  // g's ring ends before this distance
  const int kbeg = part * A.T;
  const int kend = max(kbeg, min(kbeg + A.T, (rend - A.d_lo) * kSTiles));
  sym64_tiles<E, false>(A, sh, g, kbeg, kend, A.pi + (size_t)part * E::NC * A.npad);
}

// One evaluation: staging, then per chunk of the half ring a pair kernel and a slot
// sum (component c of the sums to out, outm, outs as in sym_reduce_kernel).
template <class E>
int launch_sym64(int64_t n, const double* x, const double* m, const double* w, const double* u, double* out, double* outm,
                 double* outs, double G, double eps, bool excl, const PairConfig& cfg, hipStream_t s,
                 Sym64Kdk* step = nullptr) {
  constexpr int NC = E::NC;
  if (n == 0) return NBODY_OK;
  int nb, T, D;
  // per particle: FP64 j-side slot sums per distance, i-side sums per workgroup, the
  // slices of the blocks with themselves, and the staged records
  const int pds = diag_slices((int)((n + kSI - 1) / kSI));
  sym_plan(n, cfg.launches, NC * sizeof(double), NC * sizeof(double), NC * sizeof(double),
           pds * NC * (int)sizeof(double) + E::NR * (int)sizeof(double4), cfg.scratch ? cfg.scratch_bytes : SIZE_MAX, kFineTiles64, &nb,
           &T, &D);
  const int dmax = nb / 2;
  const int half = (nb % 2 == 0) ? 1 : 0;
  const int64_t npad = (int64_t)nb * kSI;
  const int nparts = D * kSTiles / T;
  const int nchunks = dmax > 0 ? (dmax + D - 1) / D : 0;
  // with two half-ring chunks or more and the library's own workspace, the slot sums
  // run on the side stream, and the slots come twice, so that a chunk's pair kernel
  // need not wait for the previous chunk's slot sum (with one chunk the cross-stream
  // waits cost more than the overlap gains: 15 us of a 0.15 ms evaluation at 16384)
  std::unique_lock<std::mutex> side_lk;
  SideStream* side = nchunks >= 2 && !cfg.scratch ? acquire_side_stream(s, side_lk) : nullptr;
  const int nbuf = side ? 2 : 1;
  int st = NBODY_OK;
  const size_t comp = sizeof(double) * NC * (size_t)npad;
  const size_t buf_bytes = comp * D + comp * nparts;  // one slot set: pj, then pi
  const size_t rec_bytes = sizeof(double4) * E::NR * (size_t)npad;
  char* ws = static_cast<char*>(pair_scratch(cfg, nbuf * buf_bytes + comp * pds + rec_bytes, &st));
  if (!ws) return st;
  double2* rec = reinterpret_cast<double2*>(ws + nbuf * buf_bytes + comp * pds);
  Sym64Args A;
  A.rec = rec;
  A.nb = nb; A.npad = (int)npad; A.dmax = dmax; A.half = half; A.d_lo = 1; A.T = T; A.nparts = nparts;
  A.Td = kSTiles / pds; A.ndiag = nb * pds; A.excl = excl ? 1 : 0; A.e2 = eps * eps;
  A.pj = A.pi = nullptr;
  A.pd = reinterpret_cast<double*>(ws + nbuf * buf_bytes);
  auto slots = [&](int b, Sym64Args& Q) {
    Q.pj = reinterpret_cast<double*>(ws + (size_t)b * buf_bytes);
    Q.pi = reinterpret_cast<double*>(ws + (size_t)b * buf_bytes + comp * D);
  };
  if (!step || step->staged != nbuf) {
    sym64_stage_kernel<E><<<(unsigned)((npad + 255) / 256), 256, 0, s>>>((int)n, (int)npad, x, m, w, u, rec);
    NB_LAUNCH_CHECK("sym64_stage_kernel");
  }
  KdkTail tail;
  if (step)
    tail = KdkTail{step->x,  step->v,  step->xt, reinterpret_cast<double*>(rec),
                   step->h, step->dt, step->nk, step->drift ? 1 : 0};
  if (step) step->staged = step->drift ? nbuf : 0;
  auto pair = [&](int c, int b) -> int {
    Sym64Args B = A;
    slots(b, B);
    B.d_lo = 1 + c * D;
    if (c > 0) B.ndiag = 0;  // the blocks with themselves go with the first launch
    const unsigned grid = (unsigned)B.ndiag + (dmax > 0 ? (unsigned)nb * (unsigned)nparts : 0u);
    sym64_kernel<E><<<grid, kSL, 0, s>>>(B);
    NB_LAUNCH_CHECK("sym64_kernel");
    return NBODY_OK;
  };
  auto sum = [&](int c, int b, hipStream_t rs) -> int {
    Sym64Args B = A;
    slots(b, B);
    auto red = [&](auto kdk) {
      return launch_sym_reduce<NC, double, decltype(kdk)::value>(
          n, false, nchunks >= 2, rs, (int)n, (int)npad, nb, dmax, half, 1 + c * D,
          dmax > 0 ? D : 0, dmax > 0 ? nparts : 0, B.pj, B.pi, A.pd, out, outm, G, c == 0,
          c + 1 >= nchunks, nullptr, nullptr, nullptr, nullptr, pds, outs, tail);
    };
    if constexpr (NC == 3)
      if (step) return red(std::true_type{});
    return red(std::false_type{});
  };
  if (dmax == 0) return (st = pair(0, 0)) ? st : sum(0, 0, s);
  return run_sym_chunks(side, s, nchunks, nbuf, [](hipStream_t) { return NBODY_OK; }, pair, sum);
}

}  // namespace

int launch_sym_accel64(int64_t n, const double* x, const double* m, double* a, double G, double eps, bool excl,
                       const PairConfig& cfg, hipStream_t s, Sym64Kdk* step) {
  return launch_sym64<Sym64Accel>(n, x, m, nullptr, nullptr, a, nullptr, nullptr, G, eps, excl, cfg, s, step);
}

int launch_sym_pot64(int64_t n, const double* x, const double* m, double* phi, double scale, double eps,
                     const PairConfig& cfg, hipStream_t s) {
  return launch_sym64<Sym64Pot>(n, x, m, nullptr, nullptr, phi, nullptr, nullptr, scale, eps, true, cfg, s);
}

int launch_sym_vjp64(int64_t n, const double* x, const double* m, const double* w, double* gx, double* gm, double G,
                     double eps, const PairConfig& cfg, hipStream_t s) {
  return launch_sym64<Sym64Vjp>(n, x, m, w, nullptr, gx, gm, nullptr, G, eps, true, cfg, s);
}

int launch_sym_jerk64(int64_t n, const double* x, const double* v, const double* m, double* a, double* jk, double G,
                      double eps, bool excl, const PairConfig& cfg, hipStream_t s) {
  return launch_sym64<Sym64Jerk>(n, x, m, v, nullptr, a, jk, nullptr, G, eps, excl, cfg, s);
}

int launch_sym_snap64(int64_t n, const double* x, const double* v, const double* acc, const double* m, double* a,
                      double* jk, double* sn, double G, double eps, bool excl, const PairConfig& cfg, hipStream_t s) {
  return launch_sym64<Sym64Snap>(n, x, m, v, acc, a, jk, sn, G, eps, excl, cfg, s);
}

}  // namespace nb
