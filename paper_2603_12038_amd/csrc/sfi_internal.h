// Internal declarations shared by the HIP translation units of libsfi (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sfi.h"

namespace sfi {

constexpr int kHeadDim = 128;
constexpr int kTile = 32;          // KV positions per wave iteration (two 16-row MFMA blocks)
constexpr int kWaves = 4;          // waves per attention workgroup
constexpr int kAttnThreads = 64 * kWaves;
constexpr int kStashFloats = 4096;  // per-wave LDS stash for exposed logits (16 KB): 128 / G tiles; big variant: twice that
constexpr int kMaxNmsRadius = 64;
constexpr int kSegStats = 5;        // sum f, sum r, sum f^2, sum f r, sum r^2 of one segment
constexpr int kPartStride = 132;   // floats per split record: m, l, and over J alone m, l (dense kernel), acc[128]
constexpr int kMaxSplits = 63;     // split workgroups per (sequence, KV head)
constexpr int kSlotCap = kMaxSplits + 1;  // records per (sequence, query head): one per workgroup
// Words between two arrival counters of the fast step's in-kernel merge: a cache line each.  Atomics on one line are
// performed one after the other, about 30 ns apiece.
constexpr int kArriveStride = 32;
constexpr int kSelSeg = 2048;      // Selector positions per workgroup
constexpr int kSelThreads = 256;
constexpr int kPickThreads = 1024;  // one workgroup selects for a pair (short J)
constexpr int kPickMax = 16 * kPickThreads;     // longest J it takes (16 keys per thread in registers; both sides: run_selector)
constexpr int kPickLogits = 24576;  // logits of a pair up to which it also scores
constexpr int kPriorSeg = 1024;     // positions per workgroup of the full Selector's first kernel
constexpr int kFuseThreads = 1024;   // full Selector, second kernel: workgroup ...
constexpr int kFuseSpan = 512;      // ... and positions (of every KV head) it takes
constexpr int kHistBins = 512;     // bins of a segment's coarse key histogram (long J)
constexpr int kScoreCap = 64;       // batch up to which the dense launch scores (a workgroup can meet that many sequences)
constexpr int kScorePairs = 256;    // batch times KV heads up to which it does: a workgroup per unit and pair at least
constexpr int kScoreRecords = 13;   // workgroups per sequence and KV head up to which it does ...
constexpr int kScoreRecordsFull = 8;  // ... with the full Selector
constexpr int kScoreFloats = 38400;  // LDS of a dense workgroup that scores: the waves' outputs for the combine, then their logits
constexpr int kScoreBurst = 4;       // tiles written together where a wave's part does not hold them all
__host__ __device__ constexpr int score_stash_floats(int G) { return kScoreFloats / kWaves - G * kHeadDim; }  // of a wave
__host__ __device__ constexpr int score_stay(int G, int rows) { return score_stash_floats(G) / (rows * kTile) - kScoreBurst; }  // tiles of a wave that stay in LDS
constexpr int kScoreWaitTicks = 6400;  // longest wait of a workgroup for the others of its pairs there, all sequences together (ticks of 10 ns)
constexpr int kHistGroup = 64;      // segments whose histograms a launch of its own adds up ...
constexpr int kHistGroupFrom = 128;  // ... of a J of more segments than this
constexpr int kStateWords = 8;     // per (b, h) Selector state, see SelState
constexpr int64_t kCacheBytes = (int64_t)288 << 20;  // 256 MB of last-level cache and eight L2s of 4 MB
constexpr float kNeg = -1.0e30f;   // "minus infinity" that stays finite under subtraction
constexpr float kLog2e = 1.4426950408889634f;

// Output stores: fp32, or bf16 rounded to nearest even (results here are finite: no NaN handling).
__device__ __forceinline__ uint32_t bf16_rne(float v) {
  const uint32_t u = __float_as_uint(v);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ void store_out4(float* out, int64_t elem, float4 v, bool as_bf16) {  // elem % 4 == 0
  if (as_bf16)
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + elem) =
        make_uint2(bf16_rne(v.x) | (bf16_rne(v.y) << 16), bf16_rne(v.z) | (bf16_rne(v.w) << 16));
  else
    *reinterpret_cast<float4*>(out + elem) = v;
}

// Per (sequence, KV head) Selector state words.
enum SelState { ST_BIN1 = 0, ST_K1 = 1, ST_CAND = 2 };

// A window query under the causal mask (Eq. window_logits): the query sits at row q_len - 1 of a context that ends
// at row L_end - 1, sees rows [0, q_len) only, and its evidence covers the part of the allowed set
// J = [n_sink, L_end - recent) it sees.  For the kernels that is a dense step over a context of q_len rows whose
// recent window is what is left of the real one in front of the query: rec = max(0, recent - (L_end - q_len)).
// q_len == nullptr: an ordinary step (L = L_end, rec = recent).
__device__ __forceinline__ void window_view(const int32_t* q_len, int b, int L_end, int recent, int& L, int& rec) {
  L = L_end;
  rec = recent;
  if (q_len != nullptr) {
    L = min(max(q_len[b], 0), L_end);
    rec = max(0, recent - (L_end - L));
  }
}

constexpr int kListCap = 1024;  // sequences a dense launch is planned on the device for (attn_dense_planned_kernel)

// Parameters of the full Selector's prior.
struct PriorArgs {
  float gamma, beta, p, eta, eps;
};

struct Workspace {
  float* part;        // [B*Hq][kSlotCap][kPartStride]
  float* logits;      // [B*Hq][ld_pos]   J-relative positions
  uint32_t* keys;     // [B*Hkv][ld_pos]  fp32 bit pattern of the evidence f
  uint32_t* cand;     // [B*Hkv][ld_pos][2]  keys falling into the threshold bin: the pair's list, each with its segment, or a run per segment from its
                      //   first position on, the keys alone
  uint32_t* hist;     // [B*Hkv][n_seg_cap][kHistBins / 2]  coarse key histogram of each segment, 16-bit counters
  uint32_t* state;    // [B*Hkv][kStateWords]
  uint32_t* segcnt;   // [B*Hkv][n_seg_cap]  keys of each segment in the threshold bin, and above it << 16
  int32_t* slow_list;   // [4 + 4 * B]  ragged step: the slow sequences as the dense launch planned them (see SelArgs)
  int32_t* seq_rec;     // [B]  records per query head a planned dense launch left for each sequence
  float2* jstat;      // [B*Hq]  J-only softmax statistics of each query head (slow step)
  float* prior;       // [B*Hkv][ld]  full Selector: unnormalised prior pi_kn * pi_pos
  float* fbuf;        // [B*Hkv][ld]  full Selector: evidence f
  double* segstat;    // [B*Hkv][n_seg_cap][kSegStats]  full Selector: sums for lambda* per kPriorSeg positions
  float* mu;          // [B*Hkv][ld]  windowed evidence: accumulator over the window's queries
  uint32_t* arrive;   // [B*Hkv][kWaves][kArriveStride]  workgroups of a split fast-step launch whose wave w has written its heads' records
  uint64_t* met;      // [B*Hq][kSlotCap]  scoring in the dense launch: each workgroup's statistics over J (zero between steps)
  unsigned long long* met_out;   // [B*Hkv][2]  ... mask of the records that their workgroup has left to the pair's others; workgroups counted out, and how
                                 //   many of them have left their record << 32 (zero between steps)
  int4* met_tiles;    // [B*Hkv][kSlotCap]  ... { first, step, end, - } of the tiles of the records in the mask
  uint32_t* wg_hist;  // [B*Hkv][kSlotCap][kHistBins]  ... mode 0: key histogram of each workgroup
  double* wg_stat;    // [B*Hkv][kSlotCap][kSegStats]  ... full Selector: each workgroup's sums for lambda*
  int32_t* guard;     // [1]  SFI_GUARD_* bits of device-side inputs the kernels found out of range and clamped
  int64_t ld_pos;     // multiple of kSelSeg
  int32_t n_seg_cap;
};

// Device-side inputs (lengths, counts, row indices, block ids) are clamped into the range the launch may
// touch before they address memory; a kernel that had to clamp ORs the matching bit into Workspace::guard
// once, on its way out.  The bit values are the public SFI_GUARD_* ones.
constexpr int kGuardCtxLen = 1, kGuardNSel = 2, kGuardSelIdx = 4, kGuardBlock = 8;

struct AttnArgs {
  const uint16_t* q;
  const uint16_t* K;
  const uint16_t* V;
  int64_t k_sb, k_sh, k_st, v_sb, v_sh, v_st;
  const int32_t* ctx_len;
  int32_t ms, fs;                // strides of the per-sequence entries: ctx_len / recent_start in int32, is_slow in bytes
                                 //   (1, 1 for plain arrays; 4, 16 when they are fields of a packed sfi_step_desc array)
  int32_t plan_batch;            // dense mode: > 0 = the launch plans itself on the device (attn_dense_planned_kernel); the batch
                                 //   (evidence mode with cached_rows: the sequences whose lengths add up to the launch's rows)
  int32_t plan_wgs, plan_min;    //   ... workgroups per KV head; fewest tiles a workgroup takes
  int32_t plan_even;             //   ... workgroups per pair if all sequences turn out equally long (0: do not look)
  int32_t* slow_list;            //   ... where the plan is left for the Selector's launches (see SelArgs), or nullptr
  int32_t* seq_rec;              //   ... records per query head of each sequence, [batch]
  const int32_t* q_len;          // dense and evidence mode, nullptr or: rows each sequence's query sees (window query under the causal mask)
  const int32_t* recent_start;   // gather mode
  const int32_t* sel_idx;        // gather mode
  const int32_t* n_sel;          // gather mode
  int64_t sel_stride;
  const uint8_t* is_slow;        // nullptr: every sequence takes part
  float* part;
  int32_t slot_cap;              // gather / compact mode: records each query head has room for in part (kSlotCap in a
                                 //   caller's workspace)
  int32_t cached_rows;           // evidence mode: 0 = all rows the launch may read fit the caches; else how many rows per head do
  float* logits;                 // dense mode, nullptr: do not expose logits
  uint64_t* met;                 // dense mode, nullptr or: the launch scores (score_tail); Workspace::met
  unsigned long long* met_out;   //   ... Workspace::met_out
  int4* met_tiles;               //   ... Workspace::met_tiles
  uint32_t* wg_hist;             //   ... Workspace::wg_hist
  uint32_t* keys;                //   ... Workspace::keys
  double* wg_stat;               //   ... full Selector: Workspace::wg_stat, fbuf, prior, hist, n_seg_cap, and the prior's parameters
  float* fbuf;
  float* prior;
  uint32_t* hist;
  int32_t n_seg_cap;
  float inv_alpha;
  PriorArgs prior_args;
  float alpha;                   //   ... power-mean exponent of the evidence
  int32_t met_ticks;             //   ... longest wait, in ticks of 10 ns; negative (tests): as long, and nothing is taken as arrived
  int32_t with_knorm;            // dense mode: also expose the squared key norms (full Selector)
  int32_t dense_wide;            // dense mode: K rows read as whole 128-byte lines (query groups of at most 8 heads, flat cache)
  int32_t big_stash;             // dense mode with logits: the variant with the 32 KB stash per wave (one workgroup per CU)
  float* out_direct;             // gather / compact mode with n_split == 1: write the output here, no record
  float* out_merge;              // gather / compact mode, nullptr or: the pair's last waves to finish merge the
  uint32_t* arrive;              //   pair's records into out_merge; arrive[((b * Hkv + h) * kWaves + w) * kArriveStride] counts the
                                 //   workgroups whose wave w is done (zero between launches)
  int32_t handover;              //   0: records at device scope; 1: the pair's workgroups on one XCD, records in its L2 (finish_wg);
                                 //   2: as 1, but the pair's workgroups are dealt to different XCDs
  const int32_t* table;          // paged cache: block table [B][table_stride], logical page -> block of the pool
  int64_t table_stride;
  int32_t page_lg;               // log2 of the page size in rows
  int32_t page_rpb;              // row numbers a block spans in the pool's row space (block stride / row stride)
  int64_t ld_pos;
  int32_t Hq, Hkv, G, n_sink, recent, n_split;
  int32_t max_tiles;             // dense mode: tiles of J the launch covers at most (from the host's max_len)
  int32_t row_cap;               // dense mode: max_len - 1, the last row the launch may touch
  float scale_log2;              // logit scale times log2(e): the kernels work on y = log2(e) * logit
  const uint16_t* Kc;            // compact mode: sink ++ selected rows of each (b, h), rows back to back
  const uint16_t* Vc;
  int64_t c_sb, c_sh;            // compact mode: strides between sequences / KV heads, in elements
  int32_t c_rows;                // compact mode: rows every (b, h) slice of Kc / Vc holds (all readable)
  int32_t out_bf16;              // out_direct / out_merge are bf16 (rounded to nearest even as stored), not fp32
  int32_t len_cap;               // ctx_len[b] is clamped to [0, len_cap]: the launch's max_len, else cfg.max_ctx
  int32_t n_blocks;              // paged cache: block ids are clamped to [0, n_blocks)
  int32_t* guard;                // Workspace::guard
};

// Reorg: gather the sink and the selected rows of every (b, h) into the compact buffers.
struct ReorgArgs {
  const uint16_t* K;
  const uint16_t* V;
  int64_t k_sb, k_sh, k_st, v_sb, v_sh, v_st;
  const int32_t* sel_idx;
  const int32_t* n_sel;
  const int32_t* ctx_len;
  const uint8_t* is_slow;        // nullptr: every sequence takes part
  int32_t ms, fs;                // strides of ctx_len (int32) and is_slow (bytes), see AttnArgs
  int64_t sel_stride;
  uint16_t* Kc;
  uint16_t* Vc;
  int64_t c_sb, c_sh;
  int32_t Hkv, n_sink;
  const int32_t* table;          // paged cache (see AttnArgs)
  int64_t table_stride;
  int32_t page_lg, page_rpb;
  int32_t len_cap, n_blocks;     // clamps of ctx_len and of the block ids (see AttnArgs)
  int32_t* guard;
};
constexpr int kReorgRows = 64;   // compact rows per workgroup of the Reorg kernel

struct MergeArgs {
  const float* part;
  float* out;
  const uint8_t* is_slow;
  int32_t Hq, slots_slow, slots_fast;  // slot counts for slow / fast sequences
  int32_t mode;                        // 0: all sequences use slots_slow, 1: all use slots_fast, 2: per is_slow
  float2* jstat;                       // dense records: also leave the J-only softmax statistics here (may be null)
  const int32_t* seq_rec;              // mode 0, nullptr or: records of each sequence (planned dense launch), not slots_slow
  int32_t G;                           // query heads per KV head
  float alpha;                         // power-mean exponent of the evidence (Eq. selector_mu)
  int32_t out_bf16;                    // out is bf16
  int32_t fs = 1;                      // stride of is_slow in bytes, see AttnArgs
};

struct SelArgs {
  const float2* jstat;
  const float* logits;
  uint32_t* keys;
  uint32_t* cand;
  uint32_t* hist;
  uint32_t* state;
  uint32_t* segcnt;
  const int32_t* ctx_len;
  const int32_t* q_len;    // accumulation of a window query under the causal mask (see window_view), else nullptr
  const int32_t* slow_list;  // ragged step with the planned dense launch, else nullptr: [0] number of slow sequences, then
                             //   from word 4 on { sequence, ctx_len (clamped), records per query head, 0 } for each
  const int32_t* seq_rec;  // nullptr (n_rec) or: records per query head of each sequence (planned dense launch)
  int32_t ms, fs;          // strides of ctx_len (int32) and is_slow (bytes), see AttnArgs
  const uint8_t* is_slow;
  int32_t* sel_idx;
  int32_t* n_sel;
  int64_t ld_pos;
  int32_t n_seg_cap;
  int32_t Hq, Hkv, G, n_sink, recent, budget;
  int32_t n_rec;           // dense records per query head (one per workgroup of the dense launch)
  // full Selector (mode 1)
  float* prior;
  float* fbuf;
  double* segstat;
  PriorArgs prior_args;
  float lambda_clip, alpha_soft, alpha_cross, inv_temp, eps;
  int32_t nms_radius;
  float alpha, inv_alpha;  // power-mean exponent of the evidence and its reciprocal
  // windowed evidence
  float* mu;               // [B*Hkv][ld] accumulator of the head-means of the window's queries
  float mu_scale;          // 1 / number of queries added
  int32_t accum_first;     // this query starts the accumulator
  int32_t f_from_mu;       // full Selector: take the evidence from the accumulator
  int32_t lg_rows;         // rows per tile of the exposed logits: G, or G + 1 with key norms
  // slow step in one go, mode 0: the scoring launch also merges the dense kernel's records (one more
  // workgroup per query head) and takes the J-only softmax statistics from the record headers itself
  const float* part;       // nullptr: a merge launch has run, jstat is valid
  float* merge_out;        // nullptr: nothing to merge here
  int32_t len_cap;         // the clamp the dense launch applied to ctx_len
  int32_t out_bf16;        // merge_out is bf16
  uint64_t* met;           // nullptr or: the dense launch has scored; Workspace::met
  unsigned long long* met_out;  //   ... Workspace::met_out
  const uint32_t* wg_hist;  //   ... Workspace::wg_hist (mode 0)
  const double* wg_stat;   //   ... Workspace::wg_stat (full Selector)
  int32_t place_x;         // the launch's segments lie along the grid's first index, not its second (set by the launch)
  int32_t n_place;         //   ... how many of them it has
};

hipError_t launch_attn_dense(const AttnArgs& a, int B, int n_slots, hipStream_t s);
hipError_t launch_attn_evidence(const AttnArgs& a, int B, int n_slots, hipStream_t s);  // a query of a window: logits and statistics of J
hipError_t launch_attn_dense_floor(const AttnArgs& a, int B, int n_slots, int wide, int idle_units, int writer, hipStream_t s);
hipError_t launch_attn_ragged(const AttnArgs& d, const AttnArgs& f, bool balanced, hipStream_t s);  // d: planned dense, f: gather or compact
hipError_t launch_attn_compact(const AttnArgs& a, int B, int n_slots, hipStream_t s);
hipError_t launch_reorg(const ReorgArgs& a, int B, int rows, hipStream_t s);
hipError_t launch_attn_gather(const AttnArgs& a, int B, int n_slots, hipStream_t s);
hipError_t launch_attn_gather_floor(const AttnArgs& a, int B, int n_slots, int tail, int burst, int tpw, int depth, hipStream_t s);
hipError_t launch_merge(const MergeArgs& a, int B, hipStream_t s);
// nJ: upper bound of |J|; hist: with the segments' histograms (sel_cand and sel_write follow, else sel_pick)
hipError_t launch_sel_score(SelArgs a, int B, int nJ, bool hist, hipStream_t s);
hipError_t launch_sel_accum(SelArgs a, int B, int nJ, hipStream_t s);
hipError_t launch_sel_finalize(SelArgs a, int B, int nJ, hipStream_t s);
hipError_t launch_sel_full(SelArgs a, int B, int nJ, bool hist, hipStream_t s);
bool sel_pick_scores(int nJ, int G, int pairs, int n_cu);  // whether the selecting workgroup also scores (src 1)
hipError_t launch_sel_pick(SelArgs a, int B, int nJ, int src, hipStream_t s);  // src 0: keys, 1: logits, 2: window evidence
hipError_t launch_sel_cand(SelArgs a, int B, int nJ, hipStream_t s);
hipError_t launch_sel_write(SelArgs a, int B, int nJ, hipStream_t s);
hipError_t launch_trigger(const int32_t* last_token, const uint32_t* bitmap, int vocab, int t_max, int32_t* since_slow,
                          uint8_t* is_slow, int B, hipStream_t s);
hipError_t launch_advance(int32_t* ctx_len, int32_t* recent_start, int B, int n_sink, int recent, hipStream_t s);
hipError_t launch_step_begin(sfi_step_desc* desc, const int32_t* last_token, const uint32_t* bitmap, int vocab, int t_max,
                             int advance, int B, int n_sink, int recent, hipStream_t s);

}  // namespace sfi
