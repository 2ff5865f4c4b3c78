// Sums and maxima across the lanes of a wavefront without a trip through LDS.
#pragma once
#include <hip/hip_runtime.h>

namespace ea {

// x of lane l plus x of lane l ^ 32, in every lane: one v_permlane32_swap (it hands both
// halves of the wavefront the other half's registers) instead of a trip through LDS.
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// x of lane l plus x of lane l ^ 16
__device__ __forceinline__ float sum_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// x + (x of another lane of the same 16-lane row), selected by a DPP control word
template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  int y = __builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true);
  return x + __int_as_float(y);
}

// x + (y of another lane of the same 16-lane row)
template <int CTRL>
__device__ __forceinline__ float dpp_add_of(float x, float y) {
  const int z = __builtin_amdgcn_update_dpp(0, __float_as_int(y), CTRL, 0xf, 0xf, true);
  return x + __int_as_float(z);
}

// largest of |x| in the wavefront, in every lane (x >= 0)
template <int CTRL>
__device__ __forceinline__ float dpp_max(float x) {
  return fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true)));
}
__device__ __forceinline__ float wave_max(float x) {
  x = dpp_max<0x140>(dpp_max<0x141>(dpp_max<0x4E>(dpp_max<0xB1>(x))));
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

}  // namespace ea
