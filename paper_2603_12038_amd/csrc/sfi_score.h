// The evidence of Eq. selector_mu and its coarse histogram: what the dense launch and the scoring launch have in common.
#pragma once
#include "sfi_internal.h"
#include "sfi_wave.h"

namespace sfi {

__device__ __forceinline__ float fast_exp2s(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2s(float x) { return __builtin_amdgcn_logf(x); }

// J-only softmax statistics of a head from the headers { m_J, l_J } of its dense records, one per lane (lanes without one: kNeg, 0):
// M = max of y over J; returns Z^(-alpha) / G.
__device__ __forceinline__ float group_stat(const float2 ml, float alpha, int G, float& M) {
  M = wave_max(ml.x);
  const float Z = wave_sum_f(ml.y * fast_exp2s(ml.x - M));
  const float zpow = alpha == 1.0f ? Z : fast_exp2s(alpha * fast_log2s(Z));
  return 1.0f / ((float)G * zpow);
}
__device__ __forceinline__ void add_evidence(float (&f)[4], const float4& l, float al, float M, float c) {
  f[0] += c * fast_exp2s(al * (l.x - M));
  f[1] += c * fast_exp2s(al * (l.y - M));
  f[2] += c * fast_exp2s(al * (l.z - M));
  f[3] += c * fast_exp2s(al * (l.w - M));
}
// The coarse histogram of keys: kHistBins bins of an eighth of an octave from 2^-63 up (keys outside fall into the end bins).
__device__ __forceinline__ uint32_t bin_of(uint32_t key) {
  return (uint32_t)min(max((int)(key >> 20) - (1024 - kHistBins), 0), kHistBins - 1);
}

}  // namespace sfi
