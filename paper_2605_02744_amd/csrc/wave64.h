// FP64 exchanges between the lanes of a wave.
#pragma once

#include <hip/hip_runtime.h>

namespace nb {

// A double rotated within each row of 16 lanes: lane r gets lane (r - K) mod 16's value.
template <int K>
__device__ __forceinline__ double row_ror64(double v) {
  const int l = __builtin_amdgcn_mov_dpp(__double2loint(v), 0x120 + K, 0xF, 0xF, true);
  const int h = __builtin_amdgcn_mov_dpp(__double2hiint(v), 0x120 + K, 0xF, 0xF, true);
  return __hiloint2double(h, l);
}

// Two doubles through one exchange of halves (X = 32: the wave's halves; 16: the
// odd rows of 16 lanes of a with the even rows of b), summed: lanes of the first
// kind hold a's sum over both kinds, lanes of the second kind b's.
template <int X>
__device__ __forceinline__ double swap_add(double a, double b) {
  const unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
  const unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
  if constexpr (X == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) + __hiloint2double((int)h[1], (int)l[1]);
  }
}

// Sums the M values of every lane over the wave and stores them at dst[0 .. M).
// After the two exchanges slot q of a lane in row r (of 4) holds value
// 4q + 2 (r & 1) + (r >> 1), summed over the four rows.
template <int M>
__device__ __forceinline__ void wave_sums(const double (&p)[M], double* dst) {
  const int lane = threadIdx.x & 63, row = lane >> 4;
#pragma unroll
  for (int q = 0; q < M; q += 4) {
    auto at = [&](int k) { return q + k < M ? p[q + k < M ? q + k : 0] : 0.0; };
    double v = swap_add<16>(swap_add<32>(at(0), at(1)), swap_add<32>(at(2), at(3)));
    v += row_ror64<8>(v);
    v += row_ror64<4>(v);
    v += row_ror64<2>(v);
    v += row_ror64<1>(v);
    const int k = q + 2 * (row & 1) + (row >> 1);
    if ((lane & 15) == 0 && k < M) dst[k] = v;
  }
}

// s + t rounded, its error added to e (TwoSum: exact whatever their magnitudes).
__device__ __forceinline__ double two_sum(double s, double t, double& e) {
  const double r = s + t, q = r - s;
  e += (s - (r - q)) + (t - q);
  return r;
}

// v added to the value of another lane (a DPP control that pairs lanes off), the errors
// collected in e; both lanes end up with the same.
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v, double& e) {
  auto other = [](double w) {
    const int l = __builtin_amdgcn_mov_dpp(__double2loint(w), CTRL, 0xF, 0xF, true);
    const int h = __builtin_amdgcn_mov_dpp(__double2hiint(w), CTRL, 0xF, 0xF, true);
    return __hiloint2double(h, l);
  };
  e += other(e);
  return two_sum(v, other(v), e);
}

// Sums the M values (a multiple of 4) of each of 256 lanes into tot[0 .. M): four lanes
// are added plainly by the exchanges of wave_sums, then the 64 partial sums of a value
// (part) with TwoSum by P lanes, each its share in order, then between them: quads
// (lane pairs, then the pairs of a quad), halves of a row of 16, rows.  P is what lets
// 256 lanes take all values at once.  Ends without a barrier.
template <int M>
__device__ __forceinline__ void block_sums(const double (&p)[M], double (*part)[64], double* tot) {
  static_assert(M % 4 == 0 && M <= 64, "whole rows of lanes, and four lanes a value");
  constexpr int P = M <= 16 ? 16 : M <= 32 ? 8 : 4;
  const int t = threadIdx.x, lane = t & 63, row = lane >> 4;
#pragma unroll
  for (int q = 0; q < M; q += 4)
    part[q + 2 * (row & 1) + (row >> 1)][(t >> 6) * 16 + (lane & 15)] =
        swap_add<16>(swap_add<32>(p[q], p[q + 1]), swap_add<32>(p[q + 2], p[q + 3]));
  __syncthreads();
  const int k = t / P, l = t % P;
  if (k < M) {  // the same for a value's lanes
    double v = part[k][l], e = 0.0;
#pragma unroll
    for (int w = 1; w < 64 / P; ++w) v = two_sum(v, part[k][P * w + l], e);
    v = dpp_add<0xB1>(v, e);                          // quad_perm [1, 0, 3, 2]
    v = dpp_add<0x4E>(v, e);                          // quad_perm [2, 3, 0, 1]
    if constexpr (P >= 8) v = dpp_add<0x141>(v, e);   // row_half_mirror
    if constexpr (P >= 16) v = dpp_add<0x140>(v, e);  // row_mirror
    if (l == 0) tot[k] = v + e;
  }
}

// Sums the V values of the 64 / I groups of I lanes (I = 16 or 32) into dst,
// value c of lane k of the groups at dst[c * I + k].
template <int I, int V>
__device__ __forceinline__ void group_sums(const double (&p)[V], double* dst) {
  const int lane = threadIdx.x & 63, row = lane >> 4;
  if constexpr (I == 16) {
#pragma unroll
    for (int q = 0; q < V; q += 4) {
      auto at = [&](int k) { return q + k < V ? p[q + k < V ? q + k : 0] : 0.0; };
      const double v = swap_add<16>(swap_add<32>(at(0), at(1)), swap_add<32>(at(2), at(3)));
      const int k = q + 2 * (row & 1) + (row >> 1);
      if (k < V) dst[k * I + (lane & 15)] = v;
    }
  } else {
    static_assert(I == 32, "groups of 16 or 32 lanes");
#pragma unroll
    for (int q = 0; q < V; q += 2) {
      const double v = swap_add<32>(p[q], q + 1 < V ? p[q + 1 < V ? q + 1 : 0] : 0.0);
      const int k = q + (lane >> 5);
      if (k < V) dst[k * I + (lane & 31)] = v;
    }
  }
}

// Orders a wave's LDS accesses around a rewrite by other lanes of the same wave
// (they execute in order; the compiler may otherwise move or merge them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace nb
