// Prefix sums and reductions over a 64-lane wave on the vector ALU (row shifts, half and row swaps), not the LDS crossbar.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sfi {

// Inclusive prefix sum over the 64 lanes: shifts within the rows of 16, then the row totals handed on.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
#define SFI_SCAN(ctrl, rows) v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rows, 0xf, false)
  SFI_SCAN(0x111, 0xf);  // row_shr:1
  SFI_SCAN(0x112, 0xf);  // row_shr:2
  SFI_SCAN(0x114, 0xf);  // row_shr:4
  SFI_SCAN(0x118, 0xf);  // row_shr:8
  SFI_SCAN(0x142, 0xa);  // row_bcast:15 into rows 1, 3
  SFI_SCAN(0x143, 0xc);  // row_bcast:31 into rows 2, 3
#undef SFI_SCAN
  return v;
}
// Sum over the wave, the same in every lane.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v), 63); }
template <int CTRL>
__device__ __forceinline__ float row_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// Maximum / sum of a float over the wave in every lane (fixed order).
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, row_move<0x128>(v));
  v = fmaxf(v, row_move<0x124>(v));
  v = fmaxf(v, row_move<0x122>(v));
  v = fmaxf(v, row_move<0x121>(v));
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float wave_sum_f(float v) {
  v += row_move<0x128>(v);
  v += row_move<0x124>(v);
  v += row_move<0x122>(v);
  v += row_move<0x121>(v);
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// The same for a double (two registers moved alike).
template <int CTRL>
__device__ __forceinline__ double row_move(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double wave_sum_d(double v) {
  v += row_move<0x128>(v);
  v += row_move<0x124>(v);
  v += row_move<0x122>(v);
  v += row_move<0x121>(v);
  uint64_t u = __builtin_bit_cast(uint64_t, v);
  const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  v = __builtin_bit_cast(double, (uint64_t)h[0] << 32 | l[0]) + __builtin_bit_cast(double, (uint64_t)h[1] << 32 | l[1]);
  u = __builtin_bit_cast(uint64_t, v);
  const auto l2 = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
  const auto h2 = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
  return __builtin_bit_cast(double, (uint64_t)h2[0] << 32 | l2[0]) + __builtin_bit_cast(double, (uint64_t)h2[1] << 32 | l2[1]);
}

}  // namespace sfi
