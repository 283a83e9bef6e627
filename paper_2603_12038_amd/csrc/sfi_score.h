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

// The unnormalised prior pi_kn * pi_pos of position pc (Eqs. selector_prior_kn, selector_u, selector_prior_pos) from its squared key norm.
struct Prior {
  float gamma, beta2, p, eta, eps, inv_D;
  int nJ;
  // u(j) = p / D, 1 - u(j) + eps = ((|J| - 1 - p) + eps) / D + eps with D = |J| - 1 + eps: the second
  // form keeps full relative precision near the tail, where 1 - u cancels.
  __device__ __forceinline__ Prior(const PriorArgs& a, int nJ_)
      : gamma(a.gamma), beta2(a.beta * 1.4426950408889634f), p(a.p), eta(a.eta), eps(a.eps), inv_D(1.0f / ((float)(nJ_ - 1) + a.eps)), nJ(nJ_) {}
  __device__ __forceinline__ float operator()(float k2, int pc) const {
    const float kn = -gamma * fast_log2s(sqrtf(k2) + eps);
    const float u = (float)pc * inv_D;
    const float omu = ((float)(nJ - 1 - pc) + eps) * inv_D + eps;
    const float up = u > 0.f ? fast_exp2s(p * fast_log2s(u)) : 0.f;
    const float pos = -beta2 * up + eta * fast_log2s(omu);
    return pc < nJ ? fast_exp2s(kn) * fast_exp2s(pos) : 0.f;
  }
};
// Evidence (of mu) and prior of a quad of positions added to the sums for lambda*.
__device__ __forceinline__ void add_sums(double (&sums)[kSegStats], const float (&f)[4], const float (&rr)[4]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double fd = (double)f[i], rd = (double)rr[i];
    sums[0] += fd;
    sums[1] += rd;
    sums[2] += fd * fd;
    sums[3] += fd * rd;
    sums[4] += rd * rd;
  }
}
// f = mu^(1/alpha) up to the normalisation done with the sums (Eq. selector_f); nothing past J.
__device__ __forceinline__ void evidence_of_mu(float (&f)[4], float alpha, float inv_alpha, int p, int nJ) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (alpha != 1.0f) f[i] = fast_exp2s(inv_alpha * fast_log2s(f[i]));
    f[i] = p + i < nJ ? f[i] : 0.f;
  }
}

// A quad of positions from p on, with evidence f (of mu) and squared key norms k2: keys and histogram, or (FULL) evidence and prior, added to
// the sums for lambda*.  Args: the attention launches' or the Selector's; row: the pair's first position in their arrays.
template <bool FULL, typename Args>
__device__ __forceinline__ void rank_quad(const Args& a, int64_t row, int nJ, const Prior& prior, double (&sums)[kSegStats], uint32_t* s_hist, int p,
                                          float (&f)[4], const float4& k2) {
  if (p >= nJ) return;
  if (FULL) {
    const float rr[4] = {prior(k2.x, p), prior(k2.y, p + 1), prior(k2.z, p + 2), prior(k2.w, p + 3)};
    evidence_of_mu(f, a.alpha, a.inv_alpha, p, nJ);
    add_sums(sums, f, rr);
    *reinterpret_cast<float4*>(a.fbuf + row + p) = make_float4(f[0], f[1], f[2], f[3]);
    *reinterpret_cast<float4*>(a.prior + row + p) = make_float4(rr[0], rr[1], rr[2], rr[3]);
    return;
  }
  const uint32_t key[4] = {__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]), __float_as_uint(f[3])};
  *reinterpret_cast<uint4*>(a.keys + row + p) = make_uint4(key[0], key[1], key[2], key[3]);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (p + i < nJ) atomicAdd(&s_hist[bin_of(key[i])], 1u);
}
// What a workgroup of four waves leaves of a record (slot, of its pair's kSlotCap at at): its histogram, which is put back to zero, or the sums, of every wave in
// s_sums.  Behind a barrier that follows the last rank_quad.
template <bool FULL, typename Args>
__device__ __forceinline__ void store_record_stats(const Args& a, int64_t at, uint32_t* s_hist, double (*s_sums)[kSegStats]) {
  const int tid = threadIdx.x;
  if (FULL) {
    if (tid < kSegStats) a.wg_stat[at * kSegStats + tid] = (s_sums[0][tid] + s_sums[1][tid]) + (s_sums[2][tid] + s_sums[3][tid]);
  } else {
    reinterpret_cast<uint2*>(a.wg_hist + at * kHistBins)[tid] = reinterpret_cast<const uint2*>(s_hist)[tid];
    reinterpret_cast<uint2*>(s_hist)[tid] = make_uint2(0u, 0u);
  }
}

}  // namespace sfi
