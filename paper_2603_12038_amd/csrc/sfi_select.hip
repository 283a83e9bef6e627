// Selector on the GPU (paper Algorithm 2) for gfx950.
//
// Per (sequence b, KV head h), over the allowed set J (Eq. allowed_set), positions p = j - n_sink:
//   p_g(j) = softmax over J of the logits of query head g          (Eq. selector_pt); the dense
//            kernel left y = log2(e) * logit, so e^{l - M} is 2^{y - M_y}
//   mu(j)  = (1/G) sum_g p_g(j)^alpha, f = mu^(1/alpha) / sum      (Eqs. selector_mu, selector_f; the G
//            heads of the group are the observation window; alpha = 1: f is the mean of the p_g)
// Mode 0 ranks by f alone: z = log(f + eps) is monotone in mu, so the Top-K of Eq. topk_out is taken
// on mu itself.  Mode 1 goes through the prior, the reverse-KL fusion with lambda*, Soft-NMS and the
// cross-head exclusivity first (two kernels further down) and ranks by e^z_adj.
// Top-K is a radix select on the fp32 bit pattern of the ranking value (positive floats order like unsigned integers),
// followed by an index-ordered compaction that takes every key above the threshold and the lowest-index keys
// equal to it.  Integer atomics only count, so the result does not depend on scheduling.
//
// Everything here is latency: a slow step's logits are a few MB, and what a launch costs is its chain of round trips and
// barriers.  So the number of launches follows the size of J (launch rules in sfi_api.hip):
//   one workgroup per pair does it all (sel_pick_kernel): from the logits where they are few, else from the keys that a
//   scoring launch of many workgroups has left;
//   long J: scoring with a coarse histogram per segment (stage 1; the dense launch may have done it, with a histogram
//   per workgroup: score_tail), the keys of the threshold bin collected (stage 2), the exact refinement
//   among those few keys and the compaction (stage 3), a workgroup per segment each.  The segments' histograms are added up by their readers: device-scope atomics on one cache line are
//   performed word by word, about 30 ns each, and a common histogram per pair cost a slow step 8 us (32768 positions) to
//   25 us (131072 positions, full Selector).
// In the kernels all loads that do not depend on another are requested together, uniform arguments at once, and
// prefix sums and reductions over a wave run on the vector ALU (row shifts) instead of the LDS crossbar.
#include "sfi_internal.h"
#include "sfi_merge.h"
#include "sfi_score.h"
#include "sfi_wave.h"

namespace sfi {

// ---- block primitives -----------------------------------------------------------------
// Exclusive prefix sum of one value per thread over an NT-thread block; returns the exclusive
// prefix and leaves the block total in *total.  scratch: NT / 64 words of LDS that nobody still reads.  One barrier.
template <int NT>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t* scratch, uint32_t* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t inc = wave_incl_scan(v);
  if (lane == 63) scratch[w] = inc;
  __syncthreads();
  constexpr int NW = NT / 64;
  const uint32_t t = lane < NW ? scratch[lane] : 0u;  // the waves' totals, scanned once more
  const uint32_t ti = wave_incl_scan(t);
  *total = (uint32_t)__builtin_amdgcn_readlane((int)ti, NW - 1);
  const uint32_t base = (uint32_t)__shfl((int)(ti - t), w);
  return base + inc - v;
}

// Finds, scanning bins from the highest down, the bin holding the k-th largest key (1-based k, k <= total count), with the
// thread's bins in registers: hv[i] is bin (nbins - tid * N) - 1 - i (threads past the last bin pass zeros).  Leaves
// res[0] = bin, res[1] = how many keys of that bin are still needed; valid behind the second of its two barriers.
template <int NT, int N>
__device__ __forceinline__ void find_kth_desc(const uint32_t (&hv)[N], int nbins, uint32_t k, uint32_t* res, uint32_t* scratch) {
  const int hi = nbins - (int)threadIdx.x * N;
  if (threadIdx.x == 0) res[0] = res[1] = 0u;  // defined result even if k exceeds the total
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < N; ++i) c += hv[i];
  uint32_t total;
  const uint32_t above = block_excl_scan<NT>(c, scratch, &total);
  if (above < k && k <= above + c) {
    uint32_t cum = above;
    bool found = false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if (!found && cum + hv[i] >= k) {
        res[0] = (uint32_t)(hi - 1 - i);
        res[1] = k - cum;
        found = true;
      }
      cum += hv[i];
    }
  }
  __syncthreads();
}
// The same with the histogram in LDS (N bins per thread, nbins <= NT * N).
template <int NT, int N>
__device__ __forceinline__ void find_kth_desc_lds(const uint32_t* hist, int nbins, uint32_t k, uint32_t* res, uint32_t* scratch) {
  uint32_t hv[N];
  const int hi = nbins - (int)threadIdx.x * N;
#pragma unroll
  for (int i = 0; i < N; ++i) hv[i] = hi - 1 - i >= 0 ? hist[max(hi - 1 - i, 0)] : 0u;
  find_kth_desc<NT, N>(hv, nbins, k, res, scratch);
}

// ---- which pair a workgroup works on ---------------------------------------------------------------
// LIST: the ragged step with the dense launch planned on the device.  That launch left the list of slow sequences, one record
// each { sequence, ctx_len (clamped), records per query head, - }, with their number in front; workgroups with blockIdx.z =
// r, r + gridDim.z, ... take list entries (few workgroups are launched, whatever the batch).
// Otherwise blockIdx.z is the sequence, and what does not depend on its length can be requested before the length is there.
//
// The grids' first index is the KV head (place 0, segments in the second): with eight heads, or a multiple, consecutive workgroups go
// round the eight XCDs, so all workgroups of a head, here and in the dense launch, sit behind one L2, and what
// a launch leaves for the next one -- logits, keys, histograms, candidates -- is read from there and not through the last-level cache.
// us a layer, segments first / heads first, both launches (one of them alone is worth a quarter of it): 1 x 131072 rows 102.2 / 98.6; 2 x 65536 101.2 / 97.8; 1 x 17000 29.9 / 28.8; ragged, 4 x 17000,
// one slow 37.5 / 35.2; 2 x 20000..30000, 4 KV heads 35.9 / 35.3; a query of a window over 60000 rows 26.9 / 26.3.  Where the dense work is long it is worth little: ragged, 32 x 16384..65536, two
// slow 125.9 / 125.4, 16 x 20000..60000, half slow 267.6 / 266.6, full Selector, 1 x 131071 116.9 / 116.2; with two KV heads nothing: 3 x 17000..60000 42.1 / 42.1.
// Where the second index would not do (n_place beyond kMaxPlaceY) the two change places.
struct Place {
  int head, i;  // i: segment (or what a launch has for one)
  int n;        // how many of them the launch has
};
__device__ __forceinline__ Place place_of(const SelArgs& a) {
  return a.place_x != 0 ? Place{(int)blockIdx.y, (int)blockIdx.x, a.n_place} : Place{(int)blockIdx.x, (int)blockIdx.y, a.n_place};
}
struct Cell {
  int b, bh;
  int L_in;      // ctx_len as it was read
  int n_rec;     // dense records per query head
};
template <bool LIST>
__device__ __forceinline__ int cell_count(const SelArgs& a) { return LIST ? __builtin_amdgcn_readfirstlane(a.slow_list[0]) : (int)gridDim.z; }
template <bool LIST>
__device__ __forceinline__ Cell cell_of(const SelArgs& a, int r, int head) {
  Cell c;
  if (LIST) {
    const int4 e = reinterpret_cast<const int4*>(a.slow_list)[1 + r];
    c.b = __builtin_amdgcn_readfirstlane(e.x);
    c.L_in = __builtin_amdgcn_readfirstlane(e.y);
    c.n_rec = __builtin_amdgcn_readfirstlane(e.z);
  } else {
    c.b = r;
    c.L_in = a.ctx_len[r * a.ms];
    c.n_rec = a.seq_rec != nullptr ? a.seq_rec[r] : a.n_rec;
  }
  c.bh = c.b * a.Hkv + head;
  return c;
}
// A sequence that does not take part (flags without a list: the ragged step's launch with a workgroup per cell).
template <bool LIST>
__device__ __forceinline__ bool cell_off(const SelArgs& a, const Cell& c) { return !LIST && a.is_slow != nullptr && a.is_slow[c.b * a.fs] == 0; }
__device__ __forceinline__ int nJ_of(const SelArgs& a, const Cell& c) {
  return max(0, min(c.L_in, a.len_cap) - a.recent - a.n_sink);  // the dense launch's clamp of ctx_len
}
__device__ __forceinline__ uint32_t ksel_of(const SelArgs& a, int nJ) { return (uint32_t)min(a.budget, nJ); }
// Uniform arguments every kernel here reads, asked for at once.
__device__ __forceinline__ void ask(const SelArgs& a) {
  asm volatile("" ::"s"(a.slow_list), "s"(a.ctx_len), "s"(a.is_slow), "s"(a.ms), "s"(a.fs), "s"(a.Hkv), "s"(a.len_cap), "s"(a.recent),
               "s"(a.n_sink), "s"(a.n_rec), "s"(a.seq_rec), "s"(a.ld_pos), "s"(a.keys), "s"(a.budget), "s"(a.place_x), "s"(a.n_place));
}
// Runs body(cell, thread index) for the workgroup's cells of a head; a cell's LDS is free for the next behind a barrier.
template <bool LIST, typename F>
__device__ __forceinline__ void for_cells(const SelArgs& a, int head, F body) {
  if (!LIST) {
    body(cell_of<false>(a, blockIdx.z, head), (int)threadIdx.x);
    return;
  }
  const int n = cell_count<true>(a);
  for (int r = blockIdx.z; r < n; r += gridDim.z) {
    // A zero the compiler cannot see through: without it everything a body derives from the thread index is
    // computed once in front of this loop and kept in registers across the body.
    int zero = 0;
    asm volatile("" : "+s"(zero));
    body(cell_of<true>(a, r, head), (int)threadIdx.x + zero);
    __syncthreads();
  }
}

// J-only softmax statistics of the group's heads from the headers of the dense records (one per workgroup of the dense
// launch): wave w takes heads w, w + n_waves, ..., a record per lane.  sM[g] = max of y over J, sc[g] = Z^(-alpha) / G;
// valid after the next barrier.
__device__ __forceinline__ void group_jstat(const SelArgs& a, const Cell& cell, int n_waves, float* sM, float* sc) {
  const int lane = threadIdx.x & 63;
  for (int g = threadIdx.x >> 6; g < a.G; g += n_waves) {
    const float* P = a.part + (int64_t)(cell.bh * a.G + g) * kSlotCap * kPartStride;
    const float2 ml = lane < cell.n_rec ? *reinterpret_cast<const float2*>(P + (int64_t)lane * kPartStride + 2) : make_float2(kNeg, 0.f);
    float M;
    const float c = group_stat(ml, a.alpha, a.G, M);
    if (lane == 0) {
      sM[g] = M;
      sc[g] = c;
    }
  }
}
// The slow step has no merge launch: the launch that reads the logits first carries extra workgroups that merge the dense
// records of a query head into the attention output.
__device__ __forceinline__ void merge_head(const SelArgs& a, const Cell& c, int g) {
  merge_records(a.part, a.merge_out, c.bh * a.G + g, c.n_rec, nullptr, a.G, a.alpha, a.out_bf16 != 0);
}

// Logits of (b, h): tile-major, [tile of 32 positions][rows][32], rows = the G heads (and the key norms in mode 1).
__device__ __forceinline__ float4 logits4(const float* lg, int rows, int p, int g) {
  return *reinterpret_cast<const float4*>(lg + (int64_t)(p >> 5) * (rows * kTile) + g * kTile + (p & 31));
}
// mu of NQ quads of positions p[q]: sum over heads of sc[g] 2^(alpha (y_g - sM[g])) (Eq. selector_mu).  GT >= G heads are
// loaded, all at once and without a branch; the columns past G repeat the last head and count for nothing: weight 0 and a
// maximum that makes their exponential 0 (0 times an exponential that overflowed would be NaN).  sM, sc hold GT entries.
template <int NQ, int GT>
__device__ __forceinline__ void request_logits(float4 (&lq)[NQ][GT], const float* lg, int rows, int G, const int (&p)[NQ]) {
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int g = 0; g < GT; ++g) lq[q][g] = logits4(lg, rows, p[q], min(g, G - 1));
}
template <int NQ, int GT>
__device__ __forceinline__ void evidence(float (&f)[NQ][4], const float4 (&lq)[NQ][GT], float al, const float* sM, const float* sc) {
#pragma unroll
  for (int q = 0; q < NQ; ++q)
#pragma unroll
    for (int i = 0; i < 4; ++i) f[q][i] = 0.f;
#pragma unroll
  for (int g = 0; g < GT; ++g) {
    const float M = sM[g], c = sc[g];
#pragma unroll
    for (int q = 0; q < NQ; ++q) add_evidence(f[q], lq[q][g], al, M, c);
  }
}
// The statistics of the group's heads in LDS (GT entries), from the record headers or, behind a merge launch, from jstat.
template <int GT>
__device__ __forceinline__ void group_stats(const SelArgs& a, const Cell& c, int n_waves, float* sM, float* sc) {
  const int tid = threadIdx.x;
  if (tid >= a.G && tid < GT) {
    sM[tid] = -kNeg;
    sc[tid] = 0.f;
  }
  if (a.part != nullptr) {
    group_jstat(a, c, n_waves, sM, sc);
  } else if (tid < a.G) {
    const float2 t = a.jstat[c.bh * a.G + tid];
    sM[tid] = t.x;
    sc[tid] = t.y;
  }
}

// The coarse histogram of a segment of kSelSeg keys (bin_of), two 16-bit counters per word.
__device__ __forceinline__ void hist_add4(uint32_t* s_hist, const uint32_t (&k)[4], int p, int nJ) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t bin = bin_of(k[i]);
    if (p + i < nJ) atomicAdd(&s_hist[bin >> 1], (bin & 1u) ? 0x10000u : 1u);
  }
}
__device__ __forceinline__ uint32_t* seg_hist(const SelArgs& a, int bh, int seg) {
  return a.hist + ((int64_t)bh * a.n_seg_cap + seg) * (kHistBins / 2);
}
// The sum over a group of kHistGroup segments, a word per bin.  (The pair's room holds n_seg_cap segments of kPriorSeg
// positions; segments of kSelSeg use half of it, and two places per group follow behind them.)
static_assert(kSelSeg == 2 * kPriorSeg && kHistGroup >= 4, "the groups' histograms fit behind the segments'");
__device__ __forceinline__ uint32_t* group_hist(const SelArgs& a, int bh, int grp) {
  return seg_hist(a, bh, a.n_seg_cap / 2 + 2 * grp);
}

// ---- scoring: evidence f and its key, a workgroup per NQ x 1024 positions ------------------------------
// HIST: with the segment's histogram (long J, stages 2 and 3 follow; NQ = 2: a segment per workgroup).
// ACCUM: windowed evidence (Eq. selector_mu over several queries): instead of ranking, add this
// query's head-mean to the accumulator mu (or start it, a.accum_first).
// FLAGS: flags without a list; looked at before the logits are requested, which a fast sequence does not have.  (A kernel of its own:
// the branch in front of the requests costs the slow step 0.4 us.)
template <int NQ, bool HIST, bool ACCUM, bool LIST, bool FLAGS, int GT>
__global__ __launch_bounds__(kSelThreads) void sel_score_kernel(const SelArgs a) {
  ask(a);
  asm volatile("" ::"s"(a.logits), "s"(a.lg_rows), "s"(a.part), "s"(a.G), "s"(a.alpha), "s"(a.jstat), "s"(a.merge_out));
  const Place place = place_of(a);
  const int seg = place.i;
  const int G = a.G, rows = a.lg_rows;
  __shared__ float s_jM[GT], s_jc[GT];
  __shared__ uint32_t s_hist[HIST ? kHistBins / 2 : 1];
  for_cells<LIST>(a, place.head, [&](const Cell& c, const int tid) {
    if (FLAGS && cell_off<LIST>(a, c)) return;
    const int p_lo = seg * (NQ * 1024);
    const float* lg = a.logits + (int64_t)c.bh * rows * a.ld_pos;
    int p[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) p[q] = p_lo + q * 1024 + tid * 4;
    if (a.merge_out != nullptr && seg >= place.n - G) {  // workgroup-uniform
      merge_head(a, c, seg - (place.n - G));
      return;
    }
    // (rows of logits and of the accumulator are padded to whole segments: readable whatever |J| is)
    float4 lq[NQ][GT];
    request_logits<NQ, GT>(lq, lg, rows, G, p);
    float4 m4[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      m4[q] = ACCUM && !a.accum_first ? *reinterpret_cast<const float4*>(a.mu + (int64_t)c.bh * a.ld_pos + p[q]) : make_float4(0.f, 0.f, 0.f, 0.f);
    group_stats<GT>(a, c, kSelThreads / 64, s_jM, s_jc);
    const int n_all = nJ_of(a, c);  // ACCUM under the causal mask: |J| of the whole window; nJ is the part this query sees
    int nJ = n_all;
    if (ACCUM && a.q_len != nullptr) {
      int Lq, rec;
      window_view(a.q_len, c.b, min(max(c.L_in, 0), a.len_cap), a.recent, Lq, rec);
      nJ = max(0, Lq - rec - a.n_sink);
    }
    if (ACCUM && a.accum_first && n_all > nJ) {  // the first query of a window starts the accumulator: zero where it sees nothing
      float* mu0 = a.mu + (int64_t)c.bh * a.ld_pos;
      // (from the next whole quad on: the quad that straddles the edge is written by the thread that owns it)
      for (int i = max(p_lo, (nJ + 3) & ~3) + tid; i < min(p_lo + NQ * 1024, n_all); i += kSelThreads) mu0[i] = 0.f;
    }
    if (p_lo >= nJ) return;
    static_assert(kHistBins / 2 == kSelThreads, "one word of the histogram per thread");
    if (HIST) s_hist[tid] = 0u;
    __syncthreads();  // histogram cleared, statistics in place
    float f[NQ][4];
    evidence<NQ, GT>(f, lq, a.alpha, s_jM, s_jc);
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      if (p[q] >= nJ) continue;
      if (ACCUM) {
        float4 m = m4[q];
        m.x += f[q][0];  // positions of the quad past the part this query sees take nothing from it
        m.y += p[q] + 1 < nJ ? f[q][1] : 0.f;
        m.z += p[q] + 2 < nJ ? f[q][2] : 0.f;
        m.w += p[q] + 3 < nJ ? f[q][3] : 0.f;
        *reinterpret_cast<float4*>(a.mu + (int64_t)c.bh * a.ld_pos + p[q]) = m;
        continue;
      }
      const uint32_t k[4] = {__float_as_uint(f[q][0]), __float_as_uint(f[q][1]), __float_as_uint(f[q][2]), __float_as_uint(f[q][3])};
      *reinterpret_cast<uint4*>(a.keys + (int64_t)c.bh * a.ld_pos + p[q]) = make_uint4(k[0], k[1], k[2], k[3]);
      if (HIST) hist_add4(s_hist, k, p[q], nJ);
    }
    if (HIST) {
      __syncthreads();
      seg_hist(a, c.bh, seg)[tid] = s_hist[tid];
    }
  });
}

// Windowed evidence, mode 0, long J: the accumulated mu times 1 / (number of queries added) is the ranking value.
__global__ __launch_bounds__(kSelThreads) void sel_finalize_kernel(const SelArgs a) {
  ask(a);
  const Place place = place_of(a);
  const int seg = place.i, tid = threadIdx.x;
  const Cell c = cell_of<false>(a, blockIdx.z, place.head);
  const int p_lo = seg * kSelSeg;
  const int nJ = nJ_of(a, c);
  if (p_lo >= nJ) return;
  __shared__ uint32_t s_hist[kHistBins / 2];
  uint32_t* keys = a.keys + (int64_t)c.bh * a.ld_pos;
  const float* mu = a.mu + (int64_t)c.bh * a.ld_pos;
  float4 m4[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) m4[r] = *reinterpret_cast<const float4*>(mu + p_lo + r * (kSelSeg / 2) + tid * 4);
  s_hist[tid] = 0u;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int p = p_lo + r * (kSelSeg / 2) + tid * 4;
    if (p >= nJ) continue;
    const uint32_t k[4] = {__float_as_uint(m4[r].x * a.mu_scale), __float_as_uint(m4[r].y * a.mu_scale),
                           __float_as_uint(m4[r].z * a.mu_scale), __float_as_uint(m4[r].w * a.mu_scale)};
    *reinterpret_cast<uint4*>(keys + p) = make_uint4(k[0], k[1], k[2], k[3]);
    hist_add4(s_hist, k, p, nJ);
  }
  __syncthreads();
  seg_hist(a, c.bh, seg)[tid] = s_hist[tid];
}

// ---- full Selector (mode 1): two kernels in place of the scoring --------------------------------------
// All scores of this part live in the log2 domain, Z = log2(s + eps) = z / ln 2: Soft-NMS is
// homogeneous of degree one in z, the head softmax of z / T is 2^(Z / T) normalised, and the
// adjustment alpha_cross * log(r) becomes alpha_cross * log2(r); the ranking key is 2^Z_adj = e^z_adj,
// a positive fp32 whose bit pattern orders like z_adj, so the Top-K is shared with mode 0.

// (1a) evidence f (as in mode 0) and the unnormalised prior pi_kn * pi_pos (Eqs. selector_prior_kn,
// selector_u, selector_prior_pos) of 1024 positions, and their sums for lambda*.
// FROM_MU: windowed evidence, f from the accumulator.
// FLAGS: as in the scoring kernel.
template <bool FROM_MU, bool LIST, bool FLAGS, int GT>
__global__ __launch_bounds__(kSelThreads) void sel_prior_kernel(const SelArgs a) {
  ask(a);
  asm volatile("" ::"s"(a.logits), "s"(a.part), "s"(a.G), "s"(a.alpha), "s"(a.jstat), "s"(a.prior), "s"(a.segstat), "s"(a.n_seg_cap),
               "s"(a.merge_out), "s"(a.prior_args.gamma), "s"(a.prior_args.beta), "s"(a.prior_args.p), "s"(a.prior_args.eta), "s"(a.prior_args.eps));
  const Place place = place_of(a);
  const int seg = place.i;
  const int G = a.G, rows = G + 1;
  __shared__ float s_jM[GT], s_jc[GT];
  __shared__ double s_scr[kSelThreads / 64][kSegStats];
  for_cells<LIST>(a, place.head, [&](const Cell& c, const int tid) {
    if (FLAGS && cell_off<LIST>(a, c)) return;
    if (!FROM_MU && a.merge_out != nullptr && seg >= place.n - G) {
      merge_head(a, c, seg - (place.n - G));
      return;
    }
    const int p_lo = seg * kPriorSeg;
    const int p[1] = {p_lo + tid * 4};
    const float* lg = a.logits + (int64_t)c.bh * rows * a.ld_pos;  // [tile][G heads + key norms][32]
    float4 lq[1][GT];
    float4 m4 = make_float4(0.f, 0.f, 0.f, 0.f);
    if (FROM_MU) m4 = *reinterpret_cast<const float4*>(a.mu + (int64_t)c.bh * a.ld_pos + p[0]);
    else request_logits<1, GT>(lq, lg, rows, G, p);
    const float4 k4 = logits4(lg, rows, p[0], G);
    if (!FROM_MU) group_stats<GT>(a, c, kSelThreads / 64, s_jM, s_jc);
    const int nJ = nJ_of(a, c);
    if (p_lo >= nJ) return;
    // (the next launch adds to the segments' histograms)
    if (seg % (kSelSeg / kPriorSeg) == 0) seg_hist(a, c.bh, seg / (kSelSeg / kPriorSeg))[tid] = 0u;
    const Prior prior(a.prior_args, nJ);
    const float rr[4] = {prior(k4.x, p[0]), prior(k4.y, p[0] + 1), prior(k4.z, p[0] + 2), prior(k4.w, p[0] + 3)};
    if (!FROM_MU) __syncthreads();
    float f4[1][4];
    float(&f)[4] = f4[0];
    if (FROM_MU) {  // mu was accumulated over the window's queries
      f[0] = m4.x * a.mu_scale; f[1] = m4.y * a.mu_scale; f[2] = m4.z * a.mu_scale; f[3] = m4.w * a.mu_scale;
    } else {
      evidence<1, GT>(f4, lq, a.alpha, s_jM, s_jc);
    }
    evidence_of_mu(f, a.alpha, a.inv_alpha, p[0], nJ);
    double sums[kSegStats] = {0.0, 0.0, 0.0, 0.0, 0.0};
    add_sums(sums, f, rr);
    if (p[0] < nJ) {
      *reinterpret_cast<float4*>(a.fbuf + (int64_t)c.bh * a.ld_pos + p[0]) = make_float4(f[0], f[1], f[2], f[3]);
      *reinterpret_cast<float4*>(a.prior + (int64_t)c.bh * a.ld_pos + p[0]) = make_float4(rr[0], rr[1], rr[2], rr[3]);
    }
#pragma unroll
    for (int i = 0; i < kSegStats; ++i) sums[i] = wave_sum_d(sums[i]);
    if ((tid & 63) == 0) {
#pragma unroll
      for (int i = 0; i < kSegStats; ++i) s_scr[tid >> 6][i] = sums[i];
    }
    __syncthreads();
    if (tid < kSegStats)
      a.segstat[((int64_t)c.bh * a.n_seg_cap + seg) * kSegStats + tid] = (s_scr[0][tid] + s_scr[1][tid]) + (s_scr[2][tid] + s_scr[3][tid]);
  });
}

// (1b) lambda* (Eq. selector_lambda_closed) of every KV head from its segment sums, the fused score (Eq. selector_closed),
// Z = log2(s + eps) (Eq. z_base) over the workgroup's positions and a halo of nms_radius on either side, Soft-NMS on the
// un-updated scores with the neighbourhood clipped to J (Eqs. nms_pool, nms), and the cross-head exclusivity at each
// position over the Hkv heads of the sequence (Eqs. head_softmax, head_mutex), then the ranking keys.
// A workgroup takes kFuseSpan positions of all KV heads of a sequence, eight heads at a time, so the heads' scores meet in
// LDS and no score goes to memory in between (a launch for the fusion and one for the exclusivity, each reading all heads'
// rows, took 27 us for a J of 131072 positions of 8 heads).  More than eight heads: the scores are worked out twice, once
// for the head softmax's running maximum and sum, once for the keys.
// HIST: also the heads' histograms, added to their segment's (kSelSeg / kFuseSpan workgroups share one).
// WGS: the dense launch has scored (score_tail), and the sums are its workgroups'.
template <bool HIST, bool LIST, bool WGS>
__global__ __launch_bounds__(kFuseThreads) void sel_fuse_kernel(const SelArgs a) {
  ask(a);
  if (WGS) asm volatile("" ::"s"(a.wg_stat));
  asm volatile("" ::"s"(a.fbuf), "s"(a.prior), "s"(a.segstat), "s"(a.n_seg_cap), "s"(a.nms_radius), "s"(a.eps), "s"(a.alpha_soft),
               "s"(a.alpha_cross), "s"(a.inv_temp), "s"(a.lambda_clip));
  constexpr int kGroup = 8;
  __shared__ uint32_t s_hist[HIST ? kGroup : 1][HIST ? kHistBins / 2 : 1];
  __shared__ __align__(16) float s_z[kGroup][kFuseSpan + 2 * kMaxNmsRadius];
  __shared__ __align__(16) float s_zn[kGroup][kFuseSpan];
  __shared__ float s_mx[kFuseSpan], s_sum[kFuseSpan];
  __shared__ float s_w[2][kGroup];  // weights of f and of the prior
  const int Hkv = a.Hkv, rad = a.nms_radius;
  const int zs = kFuseSpan + 2 * rad;
  for_cells<LIST>(a, 0, [&](const Cell& c, const int tid) {  // (c.bh is the sequence's first pair)
    const int lane = tid & 63, w = tid >> 6;
    const int nJ = nJ_of(a, c);
    const int p_lo = blockIdx.x * kFuseSpan;
    if (p_lo >= nJ || cell_off<LIST>(a, c)) return;
    const int n_here = min(kFuseSpan, nJ - p_lo);
    // scores after Soft-NMS of heads h0 .. h0 + nh - 1 -> s_zn
    auto scores = [&](int h0, int nh) {
      const int n_seg = WGS ? c.n_rec : (nJ + kPriorSeg - 1) / kPriorSeg;
      float fb[kGroup], pr[kGroup];  // this thread's column (position p_lo - rad + tid) of all heads, requested together
      {
        const int64_t o = (int64_t)(c.bh + h0) * a.ld_pos + min(max(p_lo - rad + tid, 0), nJ - 1);
#pragma unroll
        for (int hh = 0; hh < kGroup; ++hh) {
          fb[hh] = a.fbuf[o + (int64_t)min(hh, nh - 1) * a.ld_pos];
          pr[hh] = a.prior[o + (int64_t)min(hh, nh - 1) * a.ld_pos];
        }
      }
      if (w < nh) {  // a wave per head: lambda* in double precision, in a fixed order
        const double* st = WGS ? a.wg_stat + (int64_t)(c.bh + h0 + w) * kSlotCap * kSegStats : a.segstat + (int64_t)(c.bh + h0 + w) * a.n_seg_cap * kSegStats;
        double tot[kSegStats] = {0.0, 0.0, 0.0, 0.0, 0.0};
        for (int s0 = lane; s0 - lane < n_seg; s0 += 128) {  // two segments' sums in flight per lane
          double t0[kSegStats], t1[kSegStats];
#pragma unroll
          for (int i = 0; i < kSegStats; ++i) {
            t0[i] = st[(int64_t)min(s0, n_seg - 1) * kSegStats + i];
            t1[i] = st[(int64_t)min(s0 + 64, n_seg - 1) * kSegStats + i];
          }
#pragma unroll
          for (int i = 0; i < kSegStats; ++i) tot[i] += (s0 < n_seg ? t0[i] : 0.0) + (s0 + 64 < n_seg ? t1[i] : 0.0);
        }
#pragma unroll
        for (int i = 0; i < kSegStats; ++i) tot[i] = wave_sum_d(tot[i]);
        // f and r normalised to sum 1: |f|^2 = tot2 / F^2, f.r = tot3 / (F R), |r|^2 = tot4 / R^2
        const double iF = 1.0 / tot[0], iR = 1.0 / tot[1];
        const double ff = tot[2] * iF * iF, fr = tot[3] * iF * iR, rr = tot[4] * iR * iR;
        const double den = ff - 2.0 * fr + rr;
        double lambda = den > 1e-300 ? (ff - fr) / den : 0.0;
        lambda = fmin(fmax(lambda, 0.0), (double)a.lambda_clip);
        if (lane == 0) {
          s_w[0][w] = (float)((1.0 - lambda) * iF);
          s_w[1][w] = (float)(lambda * iR);
        }
      }
      __syncthreads();
      static_assert(kFuseSpan + 2 * kMaxNmsRadius <= kFuseThreads, "a column per thread");
      if (tid < zs) {
        const int q = p_lo - rad + tid;
#pragma unroll
        for (int hh = 0; hh < kGroup; ++hh) {
          const float z = fast_log2s(s_w[0][hh] * fb[hh] + s_w[1][hh] * pr[hh] + a.eps);
          if (hh < nh) s_z[hh][tid] = (q >= 0 && q < nJ) ? z : -INFINITY;
        }
      }
      __syncthreads();
      static_assert(kGroup * kFuseSpan == 4 * kFuseThreads, "four consecutive positions per thread");
      {
        const int hh = tid / (kFuseSpan / 4), q0 = 4 * (tid % (kFuseSpan / 4));
        const float* zc = &s_z[hh][q0];  // window of output o: zc[o .. o + 2 rad]
        if (hh < nh) {
          float m[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
          for (int e0 = 0; e0 < 2 * rad + 4; e0 += 4) {
            const float4 v4 = *reinterpret_cast<const float4*>(zc + e0);
            const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
              for (int o = 0; o < 4; ++o)
                if (e0 + k >= o && e0 + k <= o + 2 * rad) m[o] = fmaxf(m[o], v[k]);
          }
          float zn[4];
#pragma unroll
          for (int o = 0; o < 4; ++o) {
            const float z = zc[rad + o];
            zn[o] = z - a.alpha_soft * fmaxf(m[o] - z, 0.f);
          }
          *reinterpret_cast<float4*>(&s_zn[hh][q0]) = make_float4(zn[0], zn[1], zn[2], zn[3]);
        }
      }
      __syncthreads();
    };
    // cross-head softmax at each position: maximum and sum over the heads
    for (int h0 = 0; h0 < Hkv; h0 += kGroup) {
      const int nh = min(kGroup, Hkv - h0);
      scores(h0, nh);
      for (int q = tid; q < kFuseSpan; q += kFuseThreads) {
        float mx = s_zn[0][q];
        for (int hh = 1; hh < nh; ++hh) mx = fmaxf(mx, s_zn[hh][q]);
        float sum = 0.f;
        if (h0 > 0) {
          const float before = s_mx[q];
          mx = fmaxf(mx, before);
          sum = s_sum[q] * fast_exp2s((before - mx) * a.inv_temp);
        }
        for (int hh = 0; hh < nh; ++hh) sum += fast_exp2s((s_zn[hh][q] - mx) * a.inv_temp);
        s_mx[q] = mx;
        s_sum[q] = sum;
      }
      if (HIST && h0 == 0) {
        for (int i = tid; i < kGroup * kHistBins / 2; i += kFuseThreads) s_hist[i / (kHistBins / 2)][i % (kHistBins / 2)] = 0u;
      }
      __syncthreads();
    }
    const float log2_eps = fast_log2s(a.eps);
    for (int h0 = 0; h0 < Hkv; h0 += kGroup) {
      const int nh = min(kGroup, Hkv - h0);
      if (Hkv > kGroup) scores(h0, nh);
      for (int i = tid; i < nh * kFuseSpan; i += kFuseThreads) {
        const int hh = i / kFuseSpan, q = i % kFuseSpan;
        if (q < n_here) {
          const float own = s_zn[hh][q];
          // log2 of the responsibility, floored at log2(eps)
          const float lr = fmaxf((own - s_mx[q]) * a.inv_temp - fast_log2s(s_sum[q]), log2_eps);
          const uint32_t k = __float_as_uint(fast_exp2s(own + a.alpha_cross * lr));
          a.keys[(int64_t)(c.bh + h0 + hh) * a.ld_pos + p_lo + q] = k;
          if (HIST) {
            const uint32_t bin = bin_of(k);
            atomicAdd(&s_hist[hh][bin >> 1], (bin & 1u) ? 0x10000u : 1u);
          }
        }
      }
      __syncthreads();
      if (HIST) {
        for (int i = tid; i < nh * (kHistBins / 2); i += kFuseThreads) {
          const int hh = i / (kHistBins / 2), wd = i % (kHistBins / 2);
          const uint32_t v = s_hist[hh][wd];
          if (v != 0u) {
            s_hist[hh][wd] = 0u;  // for the next eight heads
            atomicAdd(&seg_hist(a, c.bh + h0 + hh, p_lo / kSelSeg)[wd], v);
          }
        }
        __syncthreads();
      }
    }
  });
}

// ---- short J: one workgroup per pair selects --------------------------------------------------------
// SRC 0: the keys a scoring launch left; 1: straight from the logits (scoring included; workgroups of places > 0 merge the
// dense records, four query heads each); 2: the accumulated evidence of a window.
// A thread holds P consecutive positions in registers.  The three radix passes run on LDS histograms over all of J;
// no list of candidates, no global histogram.
template <int P, int SRC, bool LIST, int GT>
__global__ __launch_bounds__(kPickThreads) void sel_pick_kernel(const SelArgs a) {
  ask(a);
  asm volatile("" ::"s"(a.sel_idx), "s"(a.n_sel));
  if (SRC == 1) asm volatile("" ::"s"(a.logits), "s"(a.lg_rows), "s"(a.part), "s"(a.Hq), "s"(a.G), "s"(a.alpha), "s"(a.merge_out));
  constexpr int NW = kPickThreads / 64;
  __shared__ __align__(16) uint32_t s_h[4096 + 1024 + 512];
  __shared__ uint32_t s_res[2], s_scr[4][NW];
  __shared__ float s_jM[GT], s_jc[GT];
  const Place place = place_of(a);
  for_cells<LIST>(a, place.head, [&](const Cell& c, const int tid) {
    if (cell_off<LIST>(a, c)) return;
    if (SRC == 1 && place.i > 0) {  // workgroup-uniform: one head per 256 threads
      const int g = (place.i - 1) * (kPickThreads / kMergeThreads) + (tid >> 8);
      merge_records<kPickThreads / kMergeThreads>(a.part, a.merge_out, c.bh * a.G + min(g, a.G - 1), c.n_rec, nullptr, a.G, a.alpha,
                                                  a.out_bf16 != 0, g < a.G);
      return;
    }
    const int nJ = nJ_of(a, c);
    const uint32_t ksel = ksel_of(a, nJ);
    int32_t* out = a.sel_idx + (int64_t)c.bh * a.budget;
    const int p0 = tid * P;
    uint32_t key[P];
    if (SRC == 1) {
      constexpr int NQ = P / 4;
      int p[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) p[q] = p0 + 4 * q;
      const float* lg = a.logits + (int64_t)c.bh * a.lg_rows * a.ld_pos;
      float4 lq[NQ][GT];
      if (p0 < nJ) request_logits<NQ, GT>(lq, lg, a.lg_rows, a.G, p);
      group_stats<GT>(a, c, NW, s_jM, s_jc);
      for (int i = tid; i < (4096 + 1024 + 512) / 4; i += kPickThreads) reinterpret_cast<uint4*>(s_h)[i] = make_uint4(0u, 0u, 0u, 0u);
      __syncthreads();
      float f[NQ][4];
      if (p0 < nJ) evidence<NQ, GT>(f, lq, a.alpha, s_jM, s_jc);
#pragma unroll
      for (int i = 0; i < P; ++i) key[i] = p0 + i < nJ ? __float_as_uint(f[i / 4][i % 4]) : 0u;
    } else {
      const uint32_t* src = (SRC == 0 ? a.keys : reinterpret_cast<const uint32_t*>(a.mu)) + (int64_t)c.bh * a.ld_pos;
#pragma unroll
      for (int q = 0; q < P / 4; ++q) {
        uint4 k4 = make_uint4(0u, 0u, 0u, 0u);
        if (p0 + 4 * q < nJ) k4 = *reinterpret_cast<const uint4*>(src + p0 + 4 * q);
        key[4 * q] = k4.x; key[4 * q + 1] = k4.y; key[4 * q + 2] = k4.z; key[4 * q + 3] = k4.w;
      }
      for (int i = tid; i < (4096 + 1024 + 512) / 4; i += kPickThreads) reinterpret_cast<uint4*>(s_h)[i] = make_uint4(0u, 0u, 0u, 0u);
      if (SRC == 2) {
#pragma unroll
        for (int i = 0; i < P; ++i) key[i] = __float_as_uint(__uint_as_float(key[i]) * a.mu_scale);
      }
      __syncthreads();
    }
    for (int i = (int)ksel + tid; i < a.budget; i += kPickThreads) out[i] = -1;
    if (tid == 0) a.n_sel[c.bh] = (int32_t)ksel;
    if (ksel == 0u || ksel == (uint32_t)nJ) {  // nothing, or everything
      if (ksel != 0u)
        for (int p = tid; p < nJ; p += kPickThreads) out[p] = a.n_sink + p;
      return;
    }
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (p0 + i < nJ) atomicAdd(&s_h[min(key[i] >> 19, 4095u)], 1u);
    __syncthreads();
    find_kth_desc_lds<kPickThreads, 4096 / kPickThreads>(s_h, 4096, ksel, s_res, s_scr[0]);
    const uint32_t bin1 = s_res[0], k1 = s_res[1];
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (p0 + i < nJ && (key[i] >> 19) == bin1) atomicAdd(&s_h[4096 + ((key[i] >> 9) & 1023u)], 1u);
    __syncthreads();
    find_kth_desc_lds<kPickThreads, 1>(s_h + 4096, 1024, k1, s_res, s_scr[1]);
    const uint32_t top22 = bin1 << 10 | s_res[0], k2 = s_res[1];
#pragma unroll
    for (int i = 0; i < P; ++i)
      if (p0 + i < nJ && (key[i] >> 9) == top22) atomicAdd(&s_h[4096 + 1024 + (key[i] & 511u)], 1u);
    __syncthreads();
    find_kth_desc_lds<kPickThreads, 1>(s_h + 4096 + 1024, 512, k2, s_res, s_scr[2]);
    const uint32_t tau = top22 << 9 | s_res[0], take = s_res[1];
    uint32_t cg = 0, ce = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (p0 + i < nJ) {
        cg += key[i] > tau;
        ce += key[i] == tau;
      }
    }
    uint32_t total;
    const uint32_t ex = block_excl_scan<kPickThreads>(cg | ce << 16, s_scr[3], &total);  // both at most 16384
    uint32_t gt = ex & 0xffffu, eq = ex >> 16;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      if (p0 + i < nJ) {
        const bool g = key[i] > tau, e = key[i] == tau;
        if (g || (e && eq < take)) {
          const uint32_t pos = gt + min(eq, take);
          if (pos < ksel) out[pos] = a.n_sink + p0 + i;
        }
        gt += g;
        eq += e;
      }
    }
  });
}

// ---- very long J: the segments' histograms added up by groups --------------------------------------------
// In stage 2 every segment's workgroup adds up all histograms of its pair, which grows with the square of |J|; of a J of
// more than kHistGroupFrom segments it reads the groups' sums that this launch leaves.  Both launches against stage 2
// without them, 8 pairs: 64 segments 11.2 / 8.1 us, 128 segments 12.8 / 11.9, 192 segments 13.4 / 19.6, 512 segments
// (1048576 rows) 18.0 / 84.8; 16 pairs of 128 segments 13.7 / 16.9.
template <bool LIST>
__global__ __launch_bounds__(kSelThreads) void sel_group_kernel(const SelArgs a) {
  ask(a);
  asm volatile("" ::"s"(a.hist), "s"(a.n_seg_cap));
  const Place place = place_of(a);
  const int grp = place.i;
  for_cells<LIST>(a, place.head, [&](const Cell& c, const int tid) {
    const int n_seg = (nJ_of(a, c) + kSelSeg - 1) / kSelSeg;
    const int s0 = grp * kHistGroup, s1 = min(s0 + kHistGroup, n_seg);
    if (s0 >= n_seg || cell_off<LIST>(a, c)) return;
    uint32_t lo = 0, hi = 0;
#pragma unroll 8
    for (int sg = s0; sg < s1; ++sg) {
      const uint32_t v = seg_hist(a, c.bh, sg)[tid];
      lo += v & 0xffffu;
      hi += v >> 16;
    }
    *reinterpret_cast<uint2*>(group_hist(a, c.bh, grp) + 2 * tid) = make_uint2(lo, hi);
  });
}

// ---- long J, stage 2: find the threshold bin, collect its keys ------------------------------------------
// FROM: whose histograms are added up, FROM_SEGS, FROM_GROUPS (behind sel_group_kernel) or FROM_WGS: the dense launch has
// scored, each of its workgroups (records) with a histogram of its own.  FROM_WGS, FROM_SEGS_MERGE (the full Selector behind such a
// launch): the workgroups behind the segments' merge the dense records.
enum { FROM_SEGS = 0, FROM_GROUPS = 1, FROM_WGS = 2, FROM_SEGS_MERGE = 3 };
// The candidates lie in one list per pair, each key with its segment: the segments' histograms say where a segment's part begins, and the write
// launch's threads share the list out evenly.  FROM_WGS: those histograms are not there, and each segment has a run of its own from its first position
// on, with its length in segcnt.  (Runs there too: 16 x 20000..60000 rows, half slow, write launch 8.9 -> 12.3 us; 32 x 16384..65536, two slow, 6.2 -> 8.0.)
template <bool LIST, int FROM>
__global__ __launch_bounds__(kSelThreads) void sel_cand_kernel(const SelArgs a) {
  ask(a);
  asm volatile("" ::"s"(a.state), "s"(a.hist), "s"(a.cand), "s"(a.segcnt), "s"(a.n_seg_cap));
  constexpr bool GROUPS = FROM == FROM_GROUPS, WGS = FROM == FROM_WGS, RUNS = WGS, MERGE = WGS || FROM == FROM_SEGS_MERGE;
  if (WGS) asm volatile("" ::"s"(a.wg_hist));
  if (MERGE) asm volatile("" ::"s"(a.merge_out), "s"(a.part), "s"(a.G));
  const Place place = place_of(a);
  const int seg = place.i;
  const int p_lo = seg * kSelSeg;
  __shared__ __align__(16) uint32_t s_cnt[kSelThreads / 64][kHistBins];
  __shared__ uint32_t s_res[2], s_before[kSelThreads / 64], s_all[kSelThreads / 64];
  __shared__ uint32_t s_scr[2][kSelThreads / 64];
  for_cells<LIST>(a, place.head, [&](const Cell& c, const int tid) {
    const int lane = tid & 63, w = tid >> 6;
    if (cell_off<LIST>(a, c)) return;
    if (MERGE && seg >= place.n - a.G) {  // workgroup-uniform
      merge_head(a, c, seg - (place.n - a.G));
      return;
    }
    const int nJ = nJ_of(a, c);
    const uint32_t ksel = ksel_of(a, nJ);
    const int n_seg = (nJ + kSelSeg - 1) / kSelSeg;
    if (ksel == 0u || ksel == (uint32_t)nJ || p_lo >= nJ) return;
    // The thread's 8 consecutive keys: the key row is padded to a whole segment, so both 16-byte loads are always in
    // bounds.  Then the pair's histogram: wave w adds up segments w, w + 4, ..., a lane four words (eight bins) of each.
    constexpr int kPer = kSelSeg / kSelThreads;
    static_assert(kPer == 8, "two 16-byte key loads per thread");
    const int p0 = p_lo + tid * kPer;
    uint32_t key[kPer];
    {
      const uint32_t* keys = a.keys + (int64_t)c.bh * a.ld_pos;
      const uint4 k0 = *reinterpret_cast<const uint4*>(keys + p0);
      const uint4 k1 = *reinterpret_cast<const uint4*>(keys + p0 + 4);
      key[0] = k0.x; key[1] = k0.y; key[2] = k0.z; key[3] = k0.w;
      key[4] = k1.x; key[5] = k1.y; key[6] = k1.z; key[7] = k1.w;
    }
    uint32_t cnt[8] = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
    static_assert(kHistBins == 8 * 64, "eight bins per lane");
    const int n_grp = (n_seg + kHistGroup - 1) / kHistGroup;
    if (GROUPS) {
#pragma unroll 2
      for (int gr = w; gr < n_grp; gr += kSelThreads / 64) {
        const uint4* gh = reinterpret_cast<const uint4*>(group_hist(a, c.bh, gr)) + 2 * lane;
        const uint4 q0 = gh[0], q1 = gh[1];
        cnt[0] += q0.x; cnt[1] += q0.y; cnt[2] += q0.z; cnt[3] += q0.w;
        cnt[4] += q1.x; cnt[5] += q1.y; cnt[6] += q1.z; cnt[7] += q1.w;
      }
    }
    if (WGS) {
      const uint32_t* wh = a.wg_hist + (int64_t)c.bh * kSlotCap * kHistBins;
#pragma unroll 2
      for (int sl = w; sl < c.n_rec; sl += kSelThreads / 64) {
        const uint4* gh = reinterpret_cast<const uint4*>(wh + sl * kHistBins) + 2 * lane;
        const uint4 q0 = gh[0], q1 = gh[1];
        cnt[0] += q0.x; cnt[1] += q0.y; cnt[2] += q0.z; cnt[3] += q0.w;
        cnt[4] += q1.x; cnt[5] += q1.y; cnt[6] += q1.z; cnt[7] += q1.w;
      }
    }
#pragma unroll 4
    for (int sg = w; (FROM == FROM_SEGS || FROM == FROM_SEGS_MERGE) && sg < n_seg; sg += kSelThreads / 64) {
      const uint4 q = reinterpret_cast<const uint4*>(seg_hist(a, c.bh, sg))[lane];
      cnt[0] += q.x & 0xffffu; cnt[1] += q.x >> 16; cnt[2] += q.y & 0xffffu; cnt[3] += q.y >> 16;
      cnt[4] += q.z & 0xffffu; cnt[5] += q.z >> 16; cnt[6] += q.w & 0xffffu; cnt[7] += q.w >> 16;
    }
    *reinterpret_cast<uint4*>(&s_cnt[w][8 * lane]) = make_uint4(cnt[0], cnt[1], cnt[2], cnt[3]);
    *reinterpret_cast<uint4*>(&s_cnt[w][8 * lane + 4]) = make_uint4(cnt[4], cnt[5], cnt[6], cnt[7]);
    __syncthreads();
    uint32_t hv[2];  // bins kHistBins - 1 - 2 tid and the one below
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int bin = kHistBins - 1 - 2 * tid - i;
      hv[i] = s_cnt[0][bin] + s_cnt[1][bin] + s_cnt[2][bin] + s_cnt[3][bin];
    }
    uint32_t* st = a.state + (int64_t)c.bh * kStateWords;
    find_kth_desc<kSelThreads, 2>(hv, kHistBins, ksel, s_res, s_scr[0]);
    const uint32_t bin1 = s_res[0];
    if (!RUNS) {  // candidates of the segments before this one: where this segment's part of the list begins
      uint32_t before = 0, all = 0;
      const int my_grp = seg / kHistGroup;
      for (int gr = tid; GROUPS && gr < n_grp; gr += kSelThreads) {
        const uint32_t x = group_hist(a, c.bh, gr)[bin1];
        all += x;
        before += gr < my_grp ? x : 0u;
      }
      for (int sg = (GROUPS ? my_grp * kHistGroup : 0) + tid; sg < (GROUPS ? seg : n_seg); sg += kSelThreads) {
        const uint32_t v = seg_hist(a, c.bh, sg)[bin1 >> 1];
        const uint32_t x = (bin1 & 1u) ? v >> 16 : v & 0xffffu;
        if (!GROUPS) all += x;
        before += sg < seg ? x : 0u;
      }
      before = wave_sum(before);
      all = wave_sum(all);
      if (lane == 0) {
        s_before[w] = before;
        s_all[w] = all;
      }
    }
    uint32_t mine = 0;  // bit i: key i falls into the threshold bin
    uint32_t above = 0; // keys of this thread in a higher bin: selected whatever the exact threshold is
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (p0 + i < nJ) {
        const uint32_t bin = bin_of(key[i]);
        if (bin == bin1) mine |= 1u << i;
        above += bin > bin1;
      }
    }
    // One prefix sum over the workgroup gives the segment's counts of candidates and of keys above the threshold bin (for
    // the write stage's prefix) and every thread's place among the segment's candidates.
    uint32_t total;
    const uint32_t ex = block_excl_scan<kSelThreads>((uint32_t)__popc(mine) | (above << 16), s_scr[1], &total);  // (its barrier covers s_before)
    if (tid == 0) {
      a.segcnt[(int64_t)c.bh * a.n_seg_cap + seg] = total;
      if (seg == 0) *reinterpret_cast<uint4*>(st) = make_uint4(bin1, s_res[1], RUNS ? 0u : s_all[0] + s_all[1] + s_all[2] + s_all[3], 0u);
    }
    uint2* const list = reinterpret_cast<uint2*>(a.cand) + (int64_t)c.bh * a.ld_pos;
    uint32_t* const run = a.cand + (int64_t)c.bh * a.ld_pos + p_lo;
    uint32_t at = (RUNS ? 0u : s_before[0] + s_before[1] + s_before[2] + s_before[3]) + (ex & 0xffffu);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if ((mine & (1u << i)) == 0u) continue;
      if (RUNS) run[at++] = key[i];
      else list[at++] = make_uint2(key[i], (uint32_t)seg);
    }
  });
}

// ---- long J, stage 3: exact threshold among the candidates, index-ordered write of the selected set -------
template <bool LIST, bool RUNS>
__global__ __launch_bounds__(kSelThreads) void sel_write_kernel(const SelArgs a) {
  ask(a);
  asm volatile("" ::"s"(a.state), "s"(a.cand), "s"(a.segcnt), "s"(a.n_seg_cap), "s"(a.sel_idx), "s"(a.n_sel), "s"(a.met), "s"(a.met_out));
  const Place place = place_of(a);
  const int seg = place.i;
  const int n_seg = place.n;
  __shared__ __align__(16) uint32_t s_h[2048 + 1024 + 1024];
  __shared__ uint32_t s_res[2], s_gt[kSelThreads / 64], s_eq[kSelThreads / 64], s_more[kSelThreads / 64];
  static_assert(kSelThreads == 256, "lg_grp, s_more");
  __shared__ uint32_t s_scr[4][kSelThreads / 64];
  for_cells<LIST>(a, place.head, [&](const Cell& c, const int tid) {
    if (cell_off<LIST>(a, c)) return;
    const int nJ = nJ_of(a, c);
    const uint32_t ksel = ksel_of(a, nJ);
    const int p_lo = seg * kSelSeg;
    constexpr int kPer = kSelSeg / kSelThreads;  // consecutive positions per thread
    static_assert(kPer == 8, "two 16-byte key loads per thread");
    const int p0 = p_lo + tid * kPer;
    const int64_t bh = c.bh;
    // Requested together: the state words, the thread's keys (the key row is padded to whole segments), the counts of the
    // segments before this one, and the first kSpec candidates per thread, whether or not there are so many.  RUNS: the threads go round
    // the segments in equal groups, each with the first candidates of its segment.
    constexpr int kSpec = RUNS ? 8 : 4;
    const uint4 st4 = *reinterpret_cast<const uint4*>(a.state + bh * kStateWords);
    const uint32_t* cand = a.cand + bh * a.ld_pos;
    const uint2* list = reinterpret_cast<const uint2*>(a.cand) + bh * a.ld_pos;
    const uint32_t* segcnt = a.segcnt + bh * a.n_seg_cap;
    const int lg_grp = max(0, __builtin_clz((n_seg - 1) | 1) - 24);  // log2 of the threads of a segment
    const int c_seg = min(tid >> lg_grp, n_seg - 1), c_at = tid & ((1 << lg_grp) - 1), n_spec = kSpec << lg_grp;
    uint32_t cd[RUNS ? kSpec : 1];  // candidates c_at, c_at + group, ... of the segment: a short run leaves the later rounds empty for a whole wave
    uint2 ld[RUNS ? 1 : kSpec];
    int n_cd = 0;
    if (RUNS) {
#pragma unroll
      for (int i = 0; i < kSpec; ++i) cd[RUNS ? i : 0] = cand[(int64_t)c_seg * kSelSeg + c_at + (i << lg_grp)];
      n_cd = (int)(segcnt[c_seg] & 0xffffu);
    } else {
#pragma unroll
      for (int i = 0; i < kSpec; ++i) ld[RUNS ? 0 : i] = list[tid + i * kSelThreads];
    }
    uint32_t key[kPer];
    {
      const uint32_t* keys = a.keys + bh * a.ld_pos;
      const uint4 lo4 = *reinterpret_cast<const uint4*>(keys + p0);
      const uint4 hi4 = *reinterpret_cast<const uint4*>(keys + p0 + 4);
      key[0] = lo4.x; key[1] = lo4.y; key[2] = lo4.z; key[3] = lo4.w;
      key[4] = hi4.x; key[5] = hi4.y; key[6] = hi4.z; key[7] = hi4.w;
    }
    uint32_t gt = 0, eq = 0;
    for (int sg = tid; sg < seg; sg += kSelThreads) gt += segcnt[sg] >> 16;
    int32_t* out = a.sel_idx + bh * a.budget;
    // padding and n_sel, spread over the segments' workgroups
    for (int i = (int)ksel + seg * kSelThreads + tid; i < a.budget; i += n_seg * kSelThreads) out[i] = -1;
    if (seg == 0 && tid == 0) {
      a.n_sel[bh] = (int32_t)ksel;
      if (a.met != nullptr) a.met_out[2 * bh + 1] = 0;  // (the mask is empty)
    }
    if (seg == 0 && a.met != nullptr) {  // for the next dense launch
      for (int i = tid; i < a.G * (kSlotCap / 2); i += kSelThreads) reinterpret_cast<uint4*>(a.met + bh * a.G * kSlotCap)[i] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (ksel == 0u || p_lo >= nJ) return;
    const int p_hi = min(p_lo + kSelSeg, nJ);
    if (ksel == (uint32_t)nJ) {  // everything is selected
      for (int p = p_lo + tid; p < p_hi; p += kSelThreads) out[p] = a.n_sink + p;
      return;
    }
    // Exact threshold tau and tie quota among the keys of the threshold bin (typically a few hundred): two LDS radix
    // passes, bits [19:10] then [9:0]; every workgroup of the pair does the same.  The end bins of the histogram
    // hold keys of any magnitude: a pass over bits [30:20] comes first.
    const uint32_t bin1 = st4.x;
    uint32_t k_left = st4.y, prefix = bin1 + (1024 - kHistBins);  // bits [30:20] of the threshold
    static_assert(ST_BIN1 == 0 && ST_K1 == 1 && ST_CAND == 2, "one 16-byte load");
    const bool end_bin = bin1 == 0u || bin1 == (uint32_t)kHistBins - 1u;
    const uint32_t n_list = st4.z;
    const int n_run = (nJ + kSelSeg - 1) / kSelSeg;  // segments that have a run
    const int n_first = min(n_run, kSelThreads >> lg_grp);  // segments whose first candidates are here
    if (tid >> lg_grp >= n_first) n_cd = 0;
    bool more = n_run > n_first || n_cd > n_spec;
    for (int i = tid; i < (2048 + 1024 + 1024) / 4; i += kSelThreads) reinterpret_cast<uint4*>(s_h)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (RUNS) {
      const uint64_t any = __ballot(more);
      if ((tid & 63) == 0) s_more[tid >> 6] = any != 0;
    }
    __syncthreads();
    if (RUNS) more = (s_more[0] | s_more[1] | s_more[2] | s_more[3]) != 0u;
    auto each_candidate = [&](auto f) {
      if (!RUNS) {
#pragma unroll
        for (int i = 0; i < kSpec; ++i) {
          const uint2 x = ld[RUNS ? 0 : i];
          if ((uint32_t)(tid + i * kSelThreads) < n_list) f(x.x, (int)x.y);
        }
        for (uint32_t i = tid + kSpec * kSelThreads; i < n_list; i += kSelThreads) {
          const uint2 x = list[i];
          f(x.x, (int)x.y);
        }
        return;
      }
#pragma unroll
      for (int i = 0; i < kSpec; ++i)
        if (c_at + (i << lg_grp) < n_cd) f(cd[RUNS ? i : 0], c_seg);
      if (more) {  // the rest of longer runs, kSpec candidates a thread and trip, and of the segments behind the threads'
        for (int i0 = n_spec + c_at; i0 - c_at < n_cd; i0 += n_spec) {
          uint32_t x[kSpec];
#pragma unroll
          for (int i = 0; i < kSpec; ++i) x[i] = cand[(int64_t)c_seg * kSelSeg + min(i0 + (i << lg_grp), kSelSeg - 1)];
#pragma unroll
          for (int i = 0; i < kSpec; ++i)
            if (i0 + (i << lg_grp) < n_cd) f(x[i], c_seg);
        }
        for (int sg = n_first + (tid >> 6); sg < n_run; sg += kSelThreads / 64) {
          const int n = (int)(segcnt[sg] & 0xffffu);
          for (int i = tid & 63; i < n; i += 64) f(cand[(int64_t)sg * kSelSeg + i], sg);
        }
      }
    };
    if (end_bin) {  // uniform over the pair
      each_candidate([&](uint32_t x, int) { atomicAdd(&s_h[2048 + ((x >> 20) & 2047u)], 1u); });
      __syncthreads();
      find_kth_desc_lds<kSelThreads, 8>(s_h + 2048, 2048, k_left, s_res, s_scr[3]);
      prefix = s_res[0];
      k_left = s_res[1];
      for (int i = tid; i < 1024 / 4; i += kSelThreads) reinterpret_cast<uint4*>(s_h + 2048)[i] = make_uint4(0u, 0u, 0u, 0u);
      __syncthreads();
    }
    each_candidate([&](uint32_t x, int) {
      if ((x >> 20) == prefix) atomicAdd(&s_h[(x >> 10) & 1023u], 1u);
    });
    __syncthreads();
    find_kth_desc_lds<kSelThreads, 4>(s_h, 1024, k_left, s_res, s_scr[0]);
    const uint32_t top21 = prefix << 10 | s_res[0], k2 = s_res[1];
    each_candidate([&](uint32_t x, int) {
      if ((x >> 10) == top21) atomicAdd(&s_h[1024 + (x & 1023u)], 1u);
    });
    __syncthreads();
    find_kth_desc_lds<kSelThreads, 4>(s_h + 1024, 1024, k2, s_res, s_scr[1]);
    const uint32_t tau = top21 << 10 | s_res[0];
    const uint32_t take = s_res[1];
    // keys selected in the segments before this one: those above the threshold bin (counted by stage 2)
    // plus the bin's own keys above tau; and the ties before this segment
    each_candidate([&](uint32_t x, int sg) {
      if (sg < seg) {
        gt += x > tau;
        eq += x == tau;
      }
    });
    gt = wave_sum(gt);
    eq = wave_sum(eq);
    if ((tid & 63) == 0) {
      s_gt[tid >> 6] = gt;
      s_eq[tid >> 6] = eq;
    }
    uint32_t cg = 0, ce = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (p0 + i < p_hi) {
        cg += key[i] > tau;
        ce += key[i] == tau;
      }
    }
    uint32_t total;
    const uint32_t ex = block_excl_scan<kSelThreads>(cg | (ce << 16), s_scr[2], &total);  // (its barrier covers s_gt, s_eq)
    uint32_t gt_before = s_gt[0] + s_gt[1] + s_gt[2] + s_gt[3] + (ex & 0xffffu);
    uint32_t eq_before = s_eq[0] + s_eq[1] + s_eq[2] + s_eq[3] + (ex >> 16);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      if (p0 + i < p_hi) {
        const bool g = key[i] > tau, e = key[i] == tau;
        if (g || (e && eq_before < take)) {
          const uint32_t pos = gt_before + min(eq_before, take);
          if (pos < ksel) out[pos] = a.n_sink + p0 + i;  // always true when ctx_len <= max_len held
        }
        gt_before += g;
        eq_before += e;
      }
    }
  });
}

// ---- launches -------------------------------------------------------------------------------------------
// Workgroups along z: one per sequence, or, where the slow sequences come as a list, enough for a few of them (n_wgs
// workgroups per list entry and launch).  The limit is four times what the chip holds of these kernels' workgroups (eight per
// unit): they differ in length, and with fewer the last ones walk their entries alone.  Measured on 32 sequences of 16384 to
// 65536 rows, 8 KV heads, limits of 1024 / 2048 / 4096 / 8192 / none: all slow 1312 / 1288 / 1270 / 1266 / 1264 us a step (scoring
// launch 141 / 128 / 120 / 117 / 117), 16 slow 662 / 652 / 647 / 648 / 648, 1 to 4 slow no difference; without a limit a batch
// of hundreds would launch workgroups that find nothing to do.
static unsigned z_of(const SelArgs& a, int B, int n_wgs) {
  if (a.slow_list == nullptr) return (unsigned)B;
  const int z = 8192 / (n_wgs < 1 ? 1 : n_wgs);
  return (unsigned)(z < 1 ? 1 : z > B ? B : z);
}
// The grid of n_place places (see Place).
constexpr int kMaxPlaceY = 65535;
static dim3 place_grid(SelArgs* a, int n_place, unsigned z) {
  a->place_x = n_place > kMaxPlaceY;
  a->n_place = n_place;
  return a->place_x ? dim3(n_place, a->Hkv, z) : dim3(a->Hkv, n_place, z);
}
static int ceil_seg(int nJ, int per) { return nJ > 0 ? (nJ + per - 1) / per : 1; }
// Head counts the scoring kernels are built for: the smallest that holds G.
template <int NQ, bool HIST, bool ACCUM, bool LIST, bool FLAGS>
static void launch_score_t(const SelArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(kSelThreads);
  if (a.G <= 1) hipLaunchKernelGGL((sel_score_kernel<NQ, HIST, ACCUM, LIST, FLAGS, 1>), grid, block, 0, s, a);
  else if (a.G <= 2) hipLaunchKernelGGL((sel_score_kernel<NQ, HIST, ACCUM, LIST, FLAGS, 2>), grid, block, 0, s, a);
  else if (a.G <= 4) hipLaunchKernelGGL((sel_score_kernel<NQ, HIST, ACCUM, LIST, FLAGS, 4>), grid, block, 0, s, a);
  else if (a.G <= 5) hipLaunchKernelGGL((sel_score_kernel<NQ, HIST, ACCUM, LIST, FLAGS, 5>), grid, block, 0, s, a);
  else if (a.G <= 8) hipLaunchKernelGGL((sel_score_kernel<NQ, HIST, ACCUM, LIST, FLAGS, 8>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sel_score_kernel<NQ, HIST, ACCUM, LIST, FLAGS, 16>), grid, block, 0, s, a);
}
hipError_t launch_sel_score(SelArgs a, int B, int nJ, bool hist, hipStream_t s) {
  // with the merge on board: one more workgroup per query head
  const int n_seg = ceil_seg(nJ, hist ? kSelSeg : 1024) + (a.merge_out != nullptr ? a.G : 0);
  const dim3 grid = place_grid(&a, n_seg, z_of(a, B, n_seg * a.Hkv));
  if (a.slow_list != nullptr) {
    if (hist) launch_score_t<2, true, false, true, false>(a, grid, s);
    else launch_score_t<1, false, false, true, false>(a, grid, s);
  } else if (a.is_slow != nullptr) {
    if (hist) launch_score_t<2, true, false, false, true>(a, grid, s);
    else launch_score_t<1, false, false, false, true>(a, grid, s);
  } else {
    if (hist) launch_score_t<2, true, false, false, false>(a, grid, s);
    else launch_score_t<1, false, false, false, false>(a, grid, s);
  }
  return hipGetLastError();
}
hipError_t launch_sel_accum(SelArgs a, int B, int nJ, hipStream_t s) {
  const dim3 grid = place_grid(&a, ceil_seg(nJ, 1024) + (a.merge_out != nullptr ? a.G : 0), B);
  launch_score_t<1, false, true, false, false>(a, grid, s);
  return hipGetLastError();
}
hipError_t launch_sel_finalize(SelArgs a, int B, int nJ, hipStream_t s) {
  const dim3 grid = place_grid(&a, ceil_seg(nJ, kSelSeg), B);
  hipLaunchKernelGGL(sel_finalize_kernel, grid, dim3(kSelThreads), 0, s, a);
  return hipGetLastError();
}
template <bool FROM_MU, bool LIST, bool FLAGS>
static void launch_prior_t(const SelArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(kSelThreads);
  if (FROM_MU || a.G <= 1) hipLaunchKernelGGL((sel_prior_kernel<FROM_MU, LIST, FLAGS, 1>), grid, block, 0, s, a);
  else if (a.G <= 2) hipLaunchKernelGGL((sel_prior_kernel<false, LIST, FLAGS, 2>), grid, block, 0, s, a);
  else if (a.G <= 4) hipLaunchKernelGGL((sel_prior_kernel<false, LIST, FLAGS, 4>), grid, block, 0, s, a);
  else if (a.G <= 5) hipLaunchKernelGGL((sel_prior_kernel<false, LIST, FLAGS, 5>), grid, block, 0, s, a);
  else if (a.G <= 8) hipLaunchKernelGGL((sel_prior_kernel<false, LIST, FLAGS, 8>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sel_prior_kernel<false, LIST, FLAGS, 16>), grid, block, 0, s, a);
}
hipError_t launch_sel_full(SelArgs a, int B, int nJ, bool hist, hipStream_t s) {
  const int n_span = ceil_seg(nJ, kFuseSpan);
  if (a.met != nullptr) {  // (long J, no list)
    hipLaunchKernelGGL((sel_fuse_kernel<true, false, true>), dim3(n_span, 1, B), dim3(kFuseThreads), 0, s, a);
    return hipGetLastError();
  }
  const int n_seg = ceil_seg(nJ, kPriorSeg) + (a.merge_out != nullptr ? a.G : 0);
  const dim3 grid = place_grid(&a, n_seg, z_of(a, B, n_seg * a.Hkv));
  if (a.f_from_mu) launch_prior_t<true, false, false>(a, grid, s);  // (a window's evidence is never ranked in the ragged step)
  else if (a.slow_list != nullptr) launch_prior_t<false, true, false>(a, grid, s);
  else if (a.is_slow != nullptr) launch_prior_t<false, false, true>(a, grid, s);
  else launch_prior_t<false, false, false>(a, grid, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 fgrid(n_span, 1, z_of(a, B, n_span)), fblock(kFuseThreads);
  if (a.slow_list != nullptr) {
    if (hist) hipLaunchKernelGGL((sel_fuse_kernel<true, true, false>), fgrid, fblock, 0, s, a);
    else hipLaunchKernelGGL((sel_fuse_kernel<false, true, false>), fgrid, fblock, 0, s, a);
  } else {
    if (hist) hipLaunchKernelGGL((sel_fuse_kernel<true, false, false>), fgrid, fblock, 0, s, a);
    else hipLaunchKernelGGL((sel_fuse_kernel<false, false, false>), fgrid, fblock, 0, s, a);
  }
  return hipGetLastError();
}
template <int P, bool LIST>
static void launch_pick_logits_t(const SelArgs& a, dim3 grid, hipStream_t s) {
  const dim3 block(kPickThreads);
  if (a.G <= 1) hipLaunchKernelGGL((sel_pick_kernel<P, 1, LIST, 1>), grid, block, 0, s, a);
  else if (a.G <= 2) hipLaunchKernelGGL((sel_pick_kernel<P, 1, LIST, 2>), grid, block, 0, s, a);
  else if (a.G <= 4) hipLaunchKernelGGL((sel_pick_kernel<P, 1, LIST, 4>), grid, block, 0, s, a);
  else if (P == 8 || a.G <= 5) hipLaunchKernelGGL((sel_pick_kernel<P, 1, LIST, 5>), grid, block, 0, s, a);
  else if (a.G <= 8) hipLaunchKernelGGL((sel_pick_kernel<4, 1, LIST, 8>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sel_pick_kernel<4, 1, LIST, 16>), grid, block, 0, s, a);
}
template <int SRC, bool LIST>
static void launch_pick_keys_t(const SelArgs& a, int nJ, dim3 grid, hipStream_t s) {
  const dim3 block(kPickThreads);
  if (nJ <= 4 * kPickThreads) hipLaunchKernelGGL((sel_pick_kernel<4, SRC, LIST, 1>), grid, block, 0, s, a);
  else if (nJ <= 8 * kPickThreads) hipLaunchKernelGGL((sel_pick_kernel<8, SRC, LIST, 1>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sel_pick_kernel<16, SRC, LIST, 1>), grid, block, 0, s, a);
}
// More than 4096 positions leave room for the logits of five heads in registers.  Groups of more than eight heads fill a unit
// with every 1024-thread workgroup and load columns they do not need, so where the pairs and the merging workgroups with them
// (four per pair) do not fit the chip at once, a scoring launch of small workgroups is the faster one.  Slow step, scoring here /
// in a launch before, us, 600 rows: G = 9, 64 pairs 16.5 / 19.1, 128 pairs 24.4 / 22.1, 800 pairs 131 / 95; G = 16: 19.2 / 20.5,
// 25.2 / 25.8, 118 / 106.  G = 8: 15.1 / 17.6, 18.7 / 20.9, 87.1 / 85.6.
bool sel_pick_scores(int nJ, int G, int pairs, int n_cu) {
  return (int64_t)nJ * G <= kPickLogits && nJ <= (G <= 5 ? 8 : 4) * kPickThreads && (G <= 8 || 4 * pairs <= n_cu);
}
hipError_t launch_sel_pick(SelArgs a, int B, int nJ, int src, hipStream_t s) {
  const int per_wg = kPickThreads / kMergeThreads;
  const int extra = src == 1 ? (a.G + per_wg - 1) / per_wg : 0;
  const dim3 grid = place_grid(&a, 1 + extra, z_of(a, B, (1 + extra) * a.Hkv * 4));
  const bool list = a.slow_list != nullptr;
  if (src == 1) {
    if (nJ <= 4 * kPickThreads) {
      if (list) launch_pick_logits_t<4, true>(a, grid, s);
      else launch_pick_logits_t<4, false>(a, grid, s);
    } else {
      if (list) launch_pick_logits_t<8, true>(a, grid, s);
      else launch_pick_logits_t<8, false>(a, grid, s);
    }
  } else if (src == 2) {
    launch_pick_keys_t<2, false>(a, nJ, grid, s);
  } else {
    if (list) launch_pick_keys_t<0, true>(a, nJ, grid, s);
    else launch_pick_keys_t<0, false>(a, nJ, grid, s);
  }
  return hipGetLastError();
}
static bool from_wgs(const SelArgs& a) { return a.met != nullptr && a.wg_hist != nullptr; }
hipError_t launch_sel_cand(SelArgs a, int B, int nJ, hipStream_t s) {
  const int n_seg = ceil_seg(nJ, kSelSeg);
  const bool list = a.slow_list != nullptr;
  const dim3 block(kSelThreads);
  if (a.met != nullptr) {  // (no list) one more workgroup per query head
    const dim3 grid = place_grid(&a, n_seg + a.G, z_of(a, B, (n_seg + a.G) * a.Hkv));
    if (from_wgs(a)) hipLaunchKernelGGL((sel_cand_kernel<false, FROM_WGS>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sel_cand_kernel<false, FROM_SEGS_MERGE>), grid, block, 0, s, a);
    return hipGetLastError();
  }
  const dim3 grid = place_grid(&a, n_seg, z_of(a, B, n_seg * a.Hkv));
  if (n_seg > kHistGroupFrom) {
    const int n_grp = (n_seg + kHistGroup - 1) / kHistGroup;
    SelArgs ag = a;
    const dim3 ggrid = place_grid(&ag, n_grp, z_of(a, B, n_grp * a.Hkv));
    if (list) hipLaunchKernelGGL(sel_group_kernel<true>, ggrid, block, 0, s, ag);
    else hipLaunchKernelGGL(sel_group_kernel<false>, ggrid, block, 0, s, ag);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (list) hipLaunchKernelGGL((sel_cand_kernel<true, FROM_GROUPS>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((sel_cand_kernel<false, FROM_GROUPS>), grid, block, 0, s, a);
  } else if (list) {
    hipLaunchKernelGGL((sel_cand_kernel<true, FROM_SEGS>), grid, block, 0, s, a);
  } else {
    hipLaunchKernelGGL((sel_cand_kernel<false, FROM_SEGS>), grid, block, 0, s, a);
  }
  return hipGetLastError();
}
hipError_t launch_sel_write(SelArgs a, int B, int nJ, hipStream_t s) {
  const int n_seg = ceil_seg(nJ, kSelSeg);
  const dim3 grid = place_grid(&a, n_seg, z_of(a, B, n_seg * a.Hkv));
  const dim3 block(kSelThreads);
  if (a.slow_list != nullptr) hipLaunchKernelGGL((sel_write_kernel<true, false>), grid, block, 0, s, a);
  else if (from_wgs(a)) hipLaunchKernelGGL((sel_write_kernel<false, true>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((sel_write_kernel<false, false>), grid, block, 0, s, a);
  return hipGetLastError();
}

}  // namespace sfi
