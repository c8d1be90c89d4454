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

}  // namespace nb
