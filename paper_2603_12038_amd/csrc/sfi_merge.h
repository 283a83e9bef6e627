// Merge of split records into the attention output (device function, one workgroup per output row).
#pragma once
#include "sfi_internal.h"
#include "sfi_wave.h"

namespace sfi {

constexpr int kMergeThreads = 256;
constexpr int kMergeLanes = 8;
static_assert(kSlotCap <= 64, "one record header per lane of a wave");

// out[bg, :] = sum_s 2^{m_s - M} acc_s / sum_s 2^{m_s - M} l_s over the n_slots split records of
// (sequence, query head) bg.  One workgroup of 256 threads = 8 record lanes x 32 dim quads: every
// thread owns four output dims of every eighth record, so all of a thread's loads are independent
// and in flight together.
// If jstat != nullptr the record headers also carry the statistics over the allowed set J alone (dense kernel):
// their merge gives the J-only softmax statistics of this head for the Selector (Eq. selector_pt),
// stored as jstat[bg] = { M = max of y over J, Z^(-alpha) / G } with Z = sum over J of 2^(y - M): the
// head's term of Eq. selector_mu is then p^alpha / G = (Z^(-alpha) / G) * 2^(alpha (y - M)).
// NG > 1: the workgroup has NG groups of 256 threads, each merging a row of its own (bg per group); a group with
// live = false goes along without storing anything.
template <int NG = 1>
__device__ __forceinline__ void merge_records(const float* part, float* out, int bg, int n_slots, float2* jstat,
                                              int G, float alpha, bool out_bf16, bool live = true) {
  const float* P = part + (int64_t)bg * kSlotCap * kPartStride;
  const int tid = NG == 1 ? threadIdx.x : threadIdx.x % kMergeThreads;
  const int grp = NG == 1 ? 0 : threadIdx.x / kMergeThreads;
  const int sl = tid >> 5, c = tid & 31;

  __shared__ float g_w[NG][kSlotCap];          // 2^{m_s - M}
  __shared__ float g_wl[NG][kSlotCap];         // 2^{m_s - M} l_s
  __shared__ float g_max[NG][kMergeThreads / 64];
  __shared__ float4 g_acc[NG][kMergeLanes][32];
  float* s_w = g_w[grp];
  float* s_wl = g_wl[grp];
  float* s_max = g_max[grp];
  float4(*s_acc)[32] = g_acc[grp];

  // the record headers: one per thread
  float m = kNeg, l = 0.f, mj = kNeg, lj = 0.f;
  if (tid < n_slots) {
    const float4 hd = *reinterpret_cast<const float4*>(P + tid * kPartStride);
    m = hd.x;
    l = hd.y;
    mj = jstat != nullptr ? hd.z : kNeg;
    lj = hd.w;
  }
  float M = m;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) M = fmaxf(M, __shfl_xor(M, d));
  if ((tid & 63) == 0) s_max[tid >> 6] = M;
  // meanwhile the accumulator loads of this thread's records
  constexpr int kPer = (kSlotCap + kMergeLanes - 1) / kMergeLanes;
  float4 r[kPer];
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int s = sl + i * kMergeLanes;
    r[i] = s < n_slots ? *reinterpret_cast<const float4*>(P + s * kPartStride + 4 + 4 * c) : make_float4(0.f, 0.f, 0.f, 0.f);
  }
  if (jstat != nullptr) {  // block-uniform
    // (a wave holds all record headers: kSlotCap <= 64)
    if (tid < 64) {
      // (the Selector's launches take the same statistics from the headers themselves: same order of operations)
      const float MJ = wave_max(mj);
      const float Z = wave_sum_f(lj * __builtin_amdgcn_exp2f(mj - MJ));
      const float zpow = alpha == 1.0f ? Z : __builtin_amdgcn_exp2f(alpha * __builtin_amdgcn_logf(Z));
      if (tid == 0) jstat[bg] = make_float2(MJ, 1.0f / ((float)G * zpow));
    }
  }
  __syncthreads();
  M = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  if (tid < n_slots) {
    const float wgt = __builtin_amdgcn_exp2f(m - M);
    s_w[tid] = wgt;
    s_wl[tid] = wgt * l;
  }
  __syncthreads();
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int s = sl + i * kMergeLanes;
    if (s < n_slots) {
      const float wgt = s_w[s];
      o.x += wgt * r[i].x;
      o.y += wgt * r[i].y;
      o.z += wgt * r[i].z;
      o.w += wgt * r[i].w;
    }
  }
  s_acc[sl][c] = o;
  __syncthreads();
  if (tid < 32) {
    float Z = 0.f;
    for (int s = 0; s < n_slots; ++s) Z += s_wl[s];
    float4 t = s_acc[0][tid];
#pragma unroll
    for (int j = 1; j < kMergeLanes; ++j) {
      const float4 u = s_acc[j][tid];
      t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
    const float inv = Z > 0.f ? 1.0f / Z : 0.f;
    if (out != nullptr && live)  // nullptr: only the J statistics were wanted (evidence-only pass)
      store_out4(out, (int64_t)bg * kHeadDim + 4 * tid, make_float4(t.x * inv, t.y * inv, t.z * inv, t.w * inv),
                 out_bf16);
  }
}

}  // namespace sfi
