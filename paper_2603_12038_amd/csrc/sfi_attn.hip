// Split single-query GQA attention for gfx950: dense over a position range, or gathered by index.
//
// What it computes (paper Sec. 3.1): for one (sequence b, KV head h) and the G query heads that
// share it, logits l_g(j) = scale * <q_g, k_j> over a list of positions, and the flash-style
// partial  (m, sum_j e^{l-m}, sum_j e^{l-m} v_j)  of a share of that list, in the log2 domain
// (y = log2(e) * l, weights 2^(y - m)).
//   dense  kernels (slow step, dense attention; batches with the launch planned on the device, attn_dense_planned_kernel):
//          the waves of several workgroups share the tiles of the allowed set
//          J = [n_sink, L - recent), for which y is also exposed to the Selector (Eq. window_logits,
//          W = 1), followed by the tiles of the sink and recent rows, which the Selector never ranks
//          (Eq. allowed_set).  A wave takes its J tiles first and keeps its softmax statistics at the point where
//          they end, from which the J-only normaliser of Eq. selector_pt is merged.  The four waves of a workgroup are
//          combined into one record.
//   gather kernel (fast step): the list is  sink ++ sel_idx[0:n_sel] ++ [recent_start, L)
//          (Eq. index_set_head), strided over n_split workgroups; the four waves of a workgroup
//          are combined into one record (fewer records for the merge that follows).
//   compact kernel (fast step, two-segment layout of Sec. 4.2) and the Reorg copy that feeds it.
//
// Mapping to the matrix cores.  A wave owns 32 positions per iteration, as two 16-row blocks.
//   S^T = K_blk (16 rows x 128) . Q^T (128 x 16 heads, heads >= G are zero): 4 x mfma 16x16x32 bf16
//         per block.  Lane (jg = lane/16, n = lane%16) feeds K row n, dims kblk*32 + 8*jg .. +8
//         (one 16-byte load) and gets back S[row 4*jg+i][head n], i = 0..3.
//   O   += P (16 heads x 32 rows) . V (32 rows x 128): the contraction slot (jg, i') of the PV
//         product is mapped to row 4*jg+i' of block A (i' < 4) or block B (i' >= 4), which is
//         exactly where the S^T result left this lane's probabilities, so P never crosses lanes.
//         Lane (jg, n) loads V rows 4*jg+i' at dims 8n..8n+7 (16-byte, row-contiguous across the
//         16 lanes) and issues 8 products, one per dim offset e, taking element e of each row.
//         P is split into two bf16 terms (hi + lo) so the weights keep ~16 bits.
// bf16 x bf16 products are exact in fp32, so logits differ from an fp64 evaluation only by the
// fp32 accumulation inside the matrix core.
#include <algorithm>
#include <type_traits>

#include "sfi_internal.h"
#include "sfi_merge.h"
#include "sfi_score.h"
#include "sfi_wave.h"

namespace sfi {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Byte permutes (one instruction each): the low / high halves of two dwords side by side, first argument in the low half.
__device__ __forceinline__ uint32_t pack_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }
// two fp32 -> one dword of two truncated bf16 (low half = a)
__device__ __forceinline__ uint32_t pack_hi16(float a, float b) { return pack_hi(__float_as_uint(a), __float_as_uint(b)); }

// Exchanges between the four rows of 16 lanes of a wave on the vector ALU: swapping a register with itself leaves the
// even rows' (lower half's) values twice in the first result and the odd rows' (upper half's) twice in the second.  A
// reduction over lanes n, 16 + n, 32 + n, 48 + n through the LDS crossbar is two dependent trips of about 60 ns each.
__device__ __forceinline__ float rows_max(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float t = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_sum(float v) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float t = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float half_max(float v) {
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float half_sum(float v) {
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
// Value of lane 4 * jg + I of this lane's own row of 16 (jg = its row): one row broadcast per row, each writing its row only.
template <int I>
__device__ __forceinline__ int row_quad(int v) {
  int r = __builtin_amdgcn_update_dpp(0, v, 0x150 + I, 0x1, 0xf, false);
  r = __builtin_amdgcn_update_dpp(r, v, 0x154 + I, 0x2, 0xf, false);
  r = __builtin_amdgcn_update_dpp(r, v, 0x158 + I, 0x4, 0xf, false);
  return __builtin_amdgcn_update_dpp(r, v, 0x15c + I, 0x8, 0xf, false);
}
template <int I>
__device__ __forceinline__ float row_quad(float v) { return __int_as_float(row_quad<I>(__float_as_int(v))); }

// K and V rows are read once per step: stream them past the caches (STREAM false: rows that the next launches read
// again).  base is uniform over the
// workgroup, off a 32-bit byte offset (the API rejects layouts whose per-head extent exceeds 4 GiB).
// The pieces of a row sit at constant distances (imm) behind its offset and share the one offset register.
template <bool STREAM = true>
__device__ __forceinline__ uint4 load_row16(const char* base, uint32_t off, int imm = 0) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  if (!STREAM) return *reinterpret_cast<const uint4*>(base + off + imm);
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + off + imm));
  return make_uint4(v.x, v.y, v.z, v.w);
}
// The same with a 64-bit byte offset: block pools of a paged cache may exceed 4 GiB.
template <bool STREAM = true>
__device__ __forceinline__ uint4 load_row16(const char* base, uint64_t off, int imm = 0) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  if (!STREAM) return *reinterpret_cast<const uint4*>(base + off + imm);
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + off + imm));
  return make_uint4(v.x, v.y, v.z, v.w);
}
// Offset type of a row address: 32 bits for a flat cache, 64 for a paged one.
template <bool PAGED> struct RowOff { typedef uint32_t type; };
template <> struct RowOff<true> { typedef uint64_t type; };

struct Tile {
  uint4 ka[4], kb[4];  // K rows of blocks A / B: row n, dims kblk*32 + 8*jg .. +8  (WIDE: see below)
  uint4 v[8];          // V rows 4*jg + i of block A (i < 4) and block B (i >= 4), dims 8n .. 8n+7
};

// WIDE (the gather and compact kernels, query groups of at most 8 heads): a K row's 256 bytes go out as two requests
// for whole 128-byte lines instead of four for 64 bytes -- a compute unit's bandwidth is the requests it
// keeps in flight times their size.  (The dense kernel stays with the plain layout: it measured 1-4 % slower
// with this one, whichever way the lanes exchange their halves.)  The operand layout gives a row of the matrix product to four lanes of 16 bytes, so
// a row of the product is made half a K row: the tile is four blocks of 8 positions, product row
// n = 8 * half + r of block blk is position 8 * blk + r, dims 64 * kb + 32 * half + 8 * jg .. + 8 in
// step kb (two steps), and its column 8 * half' + head is the same half of q[head].  The halves
// meet where half == half': lane (jg < 2, n < 8) and its mirror (jg + 2, n + 8), 40 lanes up.
// K registers: ka[2 * blk + kb] for blk < 2, kb[2 * (blk - 2) + kb] above.
// Position of V slot i (and of logit y[i]) of lane row jg within the tile:
template <bool WIDE>
__device__ __forceinline__ int slot_pos(int jg, int i) {
  return WIDE ? 16 * (jg >> 1) + 8 * (i >> 2) + 4 * (jg & 1) + (i & 3) : 16 * (i >> 2) + 4 * jg + (i & 3);
}
__device__ __forceinline__ uint4& wide_k(Tile& T, int blk, int kb) { return blk < 2 ? T.ka[2 * blk + kb] : T.kb[2 * (blk - 2) + kb]; }
__device__ __forceinline__ const uint4& wide_k(const Tile& T, int blk, int kb) { return blk < 2 ? T.ka[2 * blk + kb] : T.kb[2 * (blk - 2) + kb]; }
// Lane exchanges of the WIDE layout on the vector ALU (no trip through the LDS crossbar): the lane 8
// further round the same row of 16 (row rotate by 8), and the lane 40 up or down (the same, then the
// two halves of the wave swapped).
__device__ __forceinline__ int lane_xor8(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, false); }
__device__ __forceinline__ float lane_xor8(float v) { return __int_as_float(lane_xor8(__float_as_int(v))); }
__device__ __forceinline__ float lane_xor40(float v) {
  const unsigned w = (unsigned)lane_xor8(__float_as_int(v));
  const auto sw = __builtin_amdgcn_permlane32_swap(w, w, false, false);  // [0]: lower half twice, [1]: upper half twice
  return __uint_as_float((threadIdx.x & 32) != 0 ? sw[0] : sw[1]);
}
// this lane's byte offset into a K row
template <bool WIDE>
__device__ __forceinline__ uint32_t k_lane_of(int jg, int n) { return WIDE ? (uint32_t)((n >> 3) * 64 + jg * 16) : (uint32_t)(jg * 16); }

// Per-wave addressing of one (sequence, KV head): uniform bases, per-lane byte offsets.
struct Rows {
  const char* Kb;
  const char* Vb;
  uint32_t k_st, v_st;    // row strides in bytes
  uint32_t k_lane, v_lane;  // jg * 16, n * 16
  int jg, n;
};

// Paged cache: K and V are pools of blocks of 2^lg consecutive rows (row stride as in Rows); blocks
// start every rpb row strides (rpb = 2^lg when the blocks lie back to back).  A sequence's logical
// row r lives in block tbl[r >> lg] at row r & mask of that block, i.e. at row number
// tbl[r >> lg] * rpb + (r & mask) of the pool's row space.  Everything downstream of a row number
// is unchanged: kernels translate logical rows to physical ones and hand those to the same loads.
struct Pages {
  const int32_t* tbl;  // this sequence's row of the block table
  int lg, mask, rpb;
  int last;            // n_blocks - 1: a block id outside [0, last] is clamped and noted in the caller's flags
  bool live;           // ctx_len > 0 (an empty context has no valid table entry; its padding reads go to row 0 of
                       // whatever block the clamp yields and are not reported)
  __device__ __forceinline__ int page_of(int row) const { return tbl[row >> lg]; }
  __device__ __forceinline__ int phys(int row, int page, int& bad) const {
    const int pc = min(max(page, 0), last);
    bad |= (pc != page && live) ? kGuardBlock : 0;
    return pc * rpb + (row & mask);
  }
};
__device__ __forceinline__ Pages pages_of(const AttnArgs& a, int b, int L) {
  Pages P;
  P.tbl = a.table + (int64_t)b * a.table_stride;
  P.lg = a.page_lg;
  P.mask = (1 << a.page_lg) - 1;
  P.rpb = a.page_rpb;
  P.last = a.n_blocks - 1;
  P.live = L > 0;
  return P;
}

// ctx_len[b] clamped to what the launch may touch.
__device__ __forceinline__ int guarded_len(int L0, int cap, int& bad) {
  const int L = min(max(L0, 0), cap);
  bad |= L != L0 ? kGuardCtxLen : 0;
  return L;
}
// A lane that had to clamp an input says so, once, as the last thing the kernel does: a store inside the
// loop would sit in the in-order memory counter the pipelined loops wait on, and even the untaken branch,
// placed between the loop and the record write, cost the fast step 0.2 us.
__device__ __forceinline__ void report_guard(int32_t* guard, int bad) {
  if (bad != 0 && guard != nullptr) atomicOr(guard, bad);
}

// Row loads of a tile whose positions map to consecutive cache rows: block A row n is cache row
// r0 + n; rows above r_max are replaced by r_max (they carry no weight).  K and V separately, so
// that each half of the tile buffer can be refilled as soon as its consumer is done with it.
template <bool WIDE = false>
__device__ __forceinline__ void issue_k_affine(Tile& T, const Rows& R, int r0, int r_max) {
  if (WIDE) {
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      const uint32_t o = (uint32_t)min(r0 + 8 * blk + (R.n & 7), r_max) * R.k_st + R.k_lane;
      wide_k(T, blk, 0) = load_row16(R.Kb, o);
      wide_k(T, blk, 1) = load_row16(R.Kb, o, 128);
    }
    return;
  }
  const uint32_t oa = (uint32_t)min(r0 + R.n, r_max) * R.k_st + R.k_lane;
  const uint32_t ob = (uint32_t)min(r0 + 16 + R.n, r_max) * R.k_st + R.k_lane;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    T.ka[kb] = load_row16(R.Kb, oa, kb * 64);
    T.kb[kb] = load_row16(R.Kb, ob, kb * 64);
  }
}
template <bool WIDE = false>
__device__ __forceinline__ void issue_v_affine(Tile& T, const Rows& R, int r0, int r_max) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    T.v[i] = load_row16(R.Vb, (uint32_t)min(r0 + slot_pos<WIDE>(R.jg, i), r_max) * R.v_st + R.v_lane);
    T.v[4 + i] = load_row16(R.Vb, (uint32_t)min(r0 + slot_pos<WIDE>(R.jg, 4 + i), r_max) * R.v_st + R.v_lane);
  }
}
template <bool WIDE = false>
__device__ __forceinline__ void issue_affine(Tile& T, const Rows& R, int r0, int r_max) {
  issue_k_affine<WIDE>(T, R, r0, r_max);
  issue_v_affine<WIDE>(T, R, r0, r_max);
}

// Row loads of a tile with arbitrary rows: ra / rb are the cache rows of positions n and 16 + n (held by every lane of
// column n).  The other positions a lane loads are fetched from the lanes of its own row of 16 that hold them, on the
// vector ALU: a broadcast within a row of 16 per value instead of a trip through the LDS crossbar.  With 32-bit offsets the
// multiplication by the row stride happens before the exchange (once per held row, not once per load).
// OffT: RowOff<>::type.
// Value of lane I (even rows of 16) or 4 + I (odd rows) of this lane's own row of 16.
template <int I>
__device__ __forceinline__ uint32_t row_pair(uint32_t v) {
  const int r = __builtin_amdgcn_update_dpp(0, (int)v, 0x150 + I, 0x5, 0xf, false);
  return (uint32_t)__builtin_amdgcn_update_dpp(r, (int)v, 0x154 + I, 0xa, 0xf, false);
}
template <bool SCALED>
__device__ __forceinline__ uint64_t scale_row(uint32_t row, uint32_t stride) { return SCALED ? (uint64_t)row : (uint64_t)row * stride; }
template <typename OffT = uint32_t, bool WIDE = false>
__device__ __forceinline__ void issue_k_rows(Tile& T, const Rows& R, int ra, int rb) {
  constexpr bool kScaled = sizeof(OffT) == 4;
  const uint32_t a = kScaled ? (uint32_t)ra * R.k_st : (uint32_t)ra, b = kScaled ? (uint32_t)rb * R.k_st : (uint32_t)rb;
  if (WIDE) {  // positions 8 * blk + (n & 7): held by this lane or by the lane 8 further round its row of 16
    const uint32_t xa = (uint32_t)lane_xor8((int)a), xb = (uint32_t)lane_xor8((int)b);
    const bool lo = R.n < 8;
    const uint32_t r[4] = {lo ? a : xa, lo ? xa : a, lo ? b : xb, lo ? xb : b};
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      const OffT o = (OffT)(scale_row<kScaled>(r[blk], R.k_st) + R.k_lane);
      wide_k(T, blk, 0) = load_row16(R.Kb, o);
      wide_k(T, blk, 1) = load_row16(R.Kb, o, 128);
    }
    return;
  }
  const OffT oa = (OffT)(scale_row<kScaled>(a, R.k_st) + R.k_lane), ob = (OffT)(scale_row<kScaled>(b, R.k_st) + R.k_lane);
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    T.ka[kb] = load_row16(R.Kb, oa, kb * 64);
    T.kb[kb] = load_row16(R.Kb, ob, kb * 64);
  }
}
template <typename OffT = uint32_t, bool WIDE = false>
__device__ __forceinline__ void issue_v_rows(Tile& T, const Rows& R, int ra, int rb) {
  constexpr bool kScaled = sizeof(OffT) == 4;
  uint32_t r[8];
  if (WIDE) {  // slot i is position slot_pos(jg, i): index 4 * (jg & 1) + (i & 3) + 8 * (i >> 2) of ra (jg < 2) or rb
    const uint32_t row = (uint32_t)(R.jg < 2 ? ra : rb);
    const uint32_t v = kScaled ? row * R.v_st : row;
    r[0] = row_pair<0>(v); r[1] = row_pair<1>(v); r[2] = row_pair<2>(v); r[3] = row_pair<3>(v);
    r[4] = row_pair<8>(v); r[5] = row_pair<9>(v); r[6] = row_pair<10>(v); r[7] = row_pair<11>(v);
  } else {
    const int a = (int)(kScaled ? (uint32_t)ra * R.v_st : (uint32_t)ra), b = (int)(kScaled ? (uint32_t)rb * R.v_st : (uint32_t)rb);
    r[0] = row_quad<0>(a); r[1] = row_quad<1>(a); r[2] = row_quad<2>(a); r[3] = row_quad<3>(a);
    r[4] = row_quad<0>(b); r[5] = row_quad<1>(b); r[6] = row_quad<2>(b); r[7] = row_quad<3>(b);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) T.v[i] = load_row16(R.Vb, (OffT)(scale_row<kScaled>(r[i], R.v_st) + R.v_lane));
}
template <typename OffT = uint32_t, bool WIDE = false>
__device__ __forceinline__ void issue_rows(Tile& T, const Rows& R, int ra, int rb) {
  issue_k_rows<OffT, WIDE>(T, R, ra, rb);
  issue_v_rows<OffT, WIDE>(T, R, ra, rb);
}

// Q^T operand: head n, dims kblk*32 + 8*jg .. +8; columns of heads >= G read another head's row and are zeroed by mask_q
// (apart, so that nothing has to wait for q before it is needed; no branch around the loads).
// WIDE: column n = 8 * half + head holds dims 64 * kb + 32 * half + 8 * jg .. + 8 of q[head]; qreg[2], qreg[3] unused.
template <bool WIDE = false>
__device__ __forceinline__ void load_q_raw(bf16x8 (&qreg)[4], const uint16_t* q, int64_t head0, int G, int jg, int n) {
  const int head = WIDE ? n & 7 : n;
  const uint16_t* qp = q + (head0 + (head < G ? head : 0)) * kHeadDim + (WIDE ? (n >> 3) * 32 : 0) + jg * 8;
#pragma unroll
  for (int kb = 0; kb < (WIDE ? 2 : 4); ++kb) qreg[kb] = as_bf16x8(*reinterpret_cast<const uint4*>(qp + kb * (WIDE ? 64 : 32)));
}
template <bool WIDE = false>
__device__ __forceinline__ void mask_q(bf16x8 (&qreg)[4], int G, int n) {
  const uint32_t keep = (WIDE ? n & 7 : n) < G ? 0xffffffffu : 0u;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    if (WIDE && kb >= 2) {
      qreg[kb] = as_bf16x8(make_uint4(0u, 0u, 0u, 0u));
    } else {
      uint4 t = __builtin_bit_cast(uint4, qreg[kb]);
      t.x &= keep; t.y &= keep; t.z &= keep; t.w &= keep;
      qreg[kb] = as_bf16x8(t);
    }
  }
}
template <bool WIDE = false>
__device__ __forceinline__ void load_q(bf16x8 (&qreg)[4], const uint16_t* q, int64_t head0, int G, int jg, int n) {
  load_q_raw<WIDE>(qreg, q, head0, G, jg, n);
  mask_q<WIDE>(qreg, G, n);
}

// One 32-position tile in three phases: S^T = K Q^T, online softmax in the log2 domain, O += P V.
// y = c2 * <q, k> with c2 = scale * log2(e); m_run / l_run are the running max of y and the running
// sum of 2^(y - m_run) of this lane's rows; acc[e][i] is O[head 4*jg+i][dim 8n+e].
// Lanes of heads >= G see q = 0; their state stays finite and is never written out: no mask needed.

// Phase 1: y[i] = logit (log2 domain) of head n, row 4*jg+i of block A (i < 4) / block B (i >= 4).
// WIDE, first half: the eight products of a tile; after them the K registers are free for the next tile's rows.
__device__ __forceinline__ void qk_products_wide(const Tile& T, const bf16x8 (&qreg)[4], f32x4 (&s)[4]) {
#pragma unroll
  for (int blk = 0; blk < 4; ++blk) {
    s[blk] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
      s[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(wide_k(T, blk, kb)), qreg[kb], s[blk], 0, 0, 0);
  }
}
// WIDE, second half: the half-row sums meet.
// s[blk][i] of lane (jg, n): product row 4 * jg + i, column n.  Lane (jg < 2, n < 8) holds the first-half
// sums of positions 8 * blk + 4 * jg + i for head n, its mirror 40 lanes up the second-half sums.  The
// lower lane keeps blocks 0 and 1, the mirror blocks 2 and 3: each sends the other the half it lacks.
// Then lane (jg >= 2, n < 8) fetches its logits from the mirror (jg, n + 8) in its own row of 16.
__device__ __forceinline__ void qk_join_wide(const f32x4 (&s)[4], float c2, float (&y)[8]) {
  const int lane = threadIdx.x & 63, jg = lane >> 4, n = lane & 15;
  const bool low = jg < 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float u0 = (low ? s[0][i] : s[2][i]) + lane_xor40(low ? s[2][i] : s[0][i]);
    const float u1 = (low ? s[1][i] : s[3][i]) + lane_xor40(low ? s[3][i] : s[1][i]);
    const float x0 = lane_xor8(u0), x1 = lane_xor8(u1);
    y[i] = n < 8 ? (low ? u0 : x0) * c2 : 0.f;
    y[4 + i] = n < 8 ? (low ? u1 : x1) * c2 : 0.f;
  }
}

template <bool WIDE = false>
__device__ __forceinline__ void qk_phase(const Tile& T, const bf16x8 (&qreg)[4], float c2, float (&y)[8]) {
  if (WIDE) {
    f32x4 s[4];
    qk_products_wide(T, qreg, s);
    qk_join_wide(s, c2, y);
    return;
  }
  f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.ka[kb]), qreg[kb], sa, 0, 0, 0);
    sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.kb[kb]), qreg[kb], sb, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    y[i] = sa[i] * c2;
    y[4 + i] = sb[i] * c2;
  }
}

// Squared norms of the tile's K rows from the matrix cores: K K^T of block A (B), whose diagonal
// element (row m, row m) sits in lane (jg, n) = (m / 4, m), slot m % 4.  Products of bf16 pairs are
// exact in fp32.  The lane with jg == n / 4 gets ||row n||^2 of block A in k2a and of block B in k2b.
__device__ __forceinline__ void knorm_phase(const Tile& T, int jg, int n, float& k2a, float& k2b) {
  f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.ka[kb]), as_bf16x8(T.ka[kb]), sa, 0, 0, 0);
    sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(T.kb[kb]), as_bf16x8(T.kb[kb]), sb, 0, 0, 0);
  }
  const int i = n & 3;
  k2a = i == 0 ? sa[0] : i == 1 ? sa[1] : i == 2 ? sa[2] : sa[3];
  k2b = i == 0 ? sb[0] : i == 1 ? sb[1] : i == 2 ? sb[2] : sb[3];
  (void)jg;
}

// y of head n, rows 0..31 of the tile, goes to stage[n * 32 ..] (this wave's LDS patch).
template <bool WIDE = false>
__device__ __forceinline__ void stage_logits(float* stage, const float (&y)[8], int jg, int n, int G) {
  if (n < G) {
    *reinterpret_cast<float4*>(stage + n * kTile + slot_pos<WIDE>(jg, 0)) = make_float4(y[0], y[1], y[2], y[3]);
    *reinterpret_cast<float4*>(stage + n * kTile + slot_pos<WIDE>(jg, 4)) = make_float4(y[4], y[5], y[6], y[7]);
  }
}

// Ragged last tile: positions >= N carry no weight; their V rows may hold anything, so zero them
// to keep 0 * v finite.
template <bool WIDE = false>
__device__ __forceinline__ void mask_tail(Tile& T, float (&y)[8], int jg, int p0, int N) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const bool oka = p0 + slot_pos<WIDE>(jg, i) < N, okb = p0 + slot_pos<WIDE>(jg, 4 + i) < N;
    y[i] = oka ? y[i] : kNeg;
    y[4 + i] = okb ? y[4 + i] : kNeg;
    if (!oka) T.v[i] = make_uint4(0u, 0u, 0u, 0u);
    if (!okb) T.v[4 + i] = make_uint4(0u, 0u, 0u, 0u);
  }
}

// Phase 2: running max / sum update (accumulators rescaled only when some head's maximum moved,
// which is rare after the first tiles) and the weights as two bf16 terms, hi + lo ~ 16 bits.
// Masked rows carry y = kNeg; every tile handed in has at least one unmasked row, so each head's
// maximum is finite and 2^(kNeg - max) is exactly 0.
__device__ __forceinline__ void softmax_phase(const float (&y)[8], f32x4 (&acc)[8], float& m_run, float& l_run, int jg,
                                              bf16x8& a_hi, bf16x8& a_lo) {
  float mt = fmaxf(fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])), fmaxf(fmaxf(y[4], y[5]), fmaxf(y[6], y[7])));
  const float m_new = fmaxf(m_run, rows_max(mt));
  if (__ballot(m_new > m_run) != 0ull) {
    const float alpha = fast_exp2(m_run - m_new);
    l_run *= alpha;
    // this lane's accumulators belong to heads 4*jg + i
    const float al[4] = {row_quad<0>(alpha), row_quad<1>(alpha), row_quad<2>(alpha), row_quad<3>(alpha)};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[e][i] *= al[i];
    }
    m_run = m_new;
  }
  float pr[8], lo[8], ps = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    pr[i] = fast_exp2(y[i] - m_run);
    ps += pr[i];
    lo[i] = pr[i] - __uint_as_float(__float_as_uint(pr[i]) & 0xffff0000u);
  }
  l_run += ps;
  a_hi = as_bf16x8(make_uint4(pack_hi16(pr[0], pr[1]), pack_hi16(pr[2], pr[3]), pack_hi16(pr[4], pr[5]),
                              pack_hi16(pr[6], pr[7])));
  a_lo = as_bf16x8(make_uint4(pack_hi16(lo[0], lo[1]), pack_hi16(lo[2], lo[3]), pack_hi16(lo[4], lo[5]),
                              pack_hi16(lo[6], lo[7])));
}

// Phase 3: O += P V, one product per dim offset e: element e of each of the 8 rows this lane holds.
__device__ __forceinline__ void pv_phase(const Tile& T, const bf16x8& a_hi, const bf16x8& a_lo, f32x4 (&acc)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    uint32_t c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      c[i] = (e >> 1) == 0 ? T.v[i].x : (e >> 1) == 1 ? T.v[i].y : (e >> 1) == 2 ? T.v[i].z : T.v[i].w;
    const uint4 bv = (e & 1) == 0 ? make_uint4(pack_lo(c[0], c[1]), pack_lo(c[2], c[3]), pack_lo(c[4], c[5]), pack_lo(c[6], c[7]))
                                  : make_uint4(pack_hi(c[0], c[1]), pack_hi(c[2], c[3]), pack_hi(c[4], c[5]), pack_hi(c[6], c[7]));
    const bf16x8 b_e = as_bf16x8(bv);
    acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_hi, b_e, acc[e], 0, 0, 0);
    acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a_lo, b_e, acc[e], 0, 0, 0);
  }
}

// Accesses that one workgroup's records are handed to another with inside a launch, without a fence.  LOCAL false: device
// scope, visible to / from every compute unit whatever L2 it sits behind.  LOCAL true: they go to the L2 of this XCD and no
// further, visible to / from the compute units of the same XCD: the first-level caches are written through, and hold no
// older copy of a record, since its lines are read only once all workgroups have sent theirs (a launch starts with these
// caches empty; handover_for keeps the records of two heads out of one line).  They go through a buffer descriptor, 16 bytes at a time: the records of one (b, h) pair
// as a raw buffer (byte offsets, out-of-range accesses dropped by the hardware).
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
template <bool LOCAL>
constexpr int scope_bits() { return LOCAL ? 1 : 16; }  // cache-policy bits sc0, sc1 of the buffer instructions
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pair_records(float* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000);
}
template <bool LOCAL>
__device__ __forceinline__ void store_record4(__amdgpu_buffer_rsrc_t r, int byte_off, float4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)},
                                         r, byte_off, 0, scope_bits<LOCAL>());
}
template <bool LOCAL>
__device__ __forceinline__ void store_record2(__amdgpu_buffer_rsrc_t r, int byte_off, float v0, float v1) {
  __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{__float_as_uint(v0), __float_as_uint(v1)}, r, byte_off, 0, scope_bits<LOCAL>());
}
template <bool LOCAL>
__device__ __forceinline__ float4 load_record4(__amdgpu_buffer_rsrc_t r, int byte_off) {
  const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, byte_off, 0, scope_bits<LOCAL>());
  return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
template <bool LOCAL>
__device__ __forceinline__ float2 load_record2(__amdgpu_buffer_rsrc_t r, int byte_off) {
  const u32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, byte_off, 0, scope_bits<LOCAL>());
  return make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
}

// Which cell a workgroup of a fast-step launch takes.  LOCAL: the grid is laid out so that all workgroups of a pair have the
// same linear index modulo 8, and consecutive indices go round the eight XCDs: blockIdx = (pair in the row, slot, row) with
// max(8, Hkv) pairs in a row.  shape: Hkv | log2 of the metadata stride << 16 | is_slow given << 20 |
// log2 of the sequences in a row << 21 | log2 of Hkv, or 31 where a row is one sequence << 23 | pairs in a row that is not full, or 0 << 28.
// (Tests: a ninth workgroup to each row of eight, without a pair, sends a pair's slots to different XCDs.)
struct FastCell {
  int slot, h, b;
  bool off;  // no pair behind this workgroup
};
template <bool LOCAL>
__device__ __forceinline__ FastCell fast_cell(uint32_t shape) {
  if (!LOCAL) return FastCell{(int)blockIdx.x, (int)blockIdx.y, (int)blockIdx.z, false};
  const uint32_t x = blockIdx.x, lg = (shape >> 23) & 31u, np = shape >> 28, q = x >> lg;
  return FastCell{(int)blockIdx.y, (int)(x - (q << lg)), (int)((blockIdx.z << ((shape >> 21) & 3u)) + q), np != 0u && x >= np};
}

// Where an attention workgroup's result goes.
struct WgOut {
  float* out_direct;   // the workgroup is the only one of its (b, h) pair: it writes O / l straight to out[b, head, :]
  float* out_merge;    // or: records go out in stores that the pair's other workgroups can see and the last waves to finish merge them into this;
  uint32_t* arrive;    //   arrive[w * kArriveStride] counts the pair's workgroups whose wave w has sent its heads' records
  float* part;         // the records (with neither pointer above: a merge launch follows)
  int n_split, slot_cap;
  bool out_bf16;
  uint64_t* met;       // JSTAT 2: the pair's statistics for score_tail, [G][kSlotCap]
};
__device__ __forceinline__ WgOut wg_out_of(const AttnArgs& a, int bh) {
  WgOut o;
  o.out_direct = a.out_direct;
  o.out_merge = a.out_merge;
  o.arrive = a.arrive != nullptr ? a.arrive + (int64_t)bh * kWaves * kArriveStride : nullptr;
  o.part = a.part;
  o.n_split = a.n_split;
  o.slot_cap = a.slot_cap;
  o.out_bf16 = a.out_bf16 != 0;
  o.met = nullptr;
  return o;
}
// The way out of an attention workgroup: the four waves' partial results are combined through LDS and sent where WgOut
// says, and, in a split launch, the records of the pair's workgroups are merged in the kernel:
//   out[b, head, :] = sum_s 2^(m_s - M) acc_s / sum_s 2^(m_s - M) l_s.
// This is the launch's critical path (a third of a short fast step), so it is one barrier long.  Every wave leaves its
// raw partial result in LDS; behind the barrier wave w finishes the heads w, w + 4, ... by itself: it combines the four
// waves' parts (lanes 0..31 one head, 32..63 the head four further on, four output dims per lane), stores the
// workgroup's record of those heads, waits for their acknowledgement and counts itself in on the
// pair's counter for wave w.  The wave that finds all n_split - 1 others counted merges the records of its heads (even
// records in lanes 0..31, odd ones in lanes 32..63, sixteen records in flight) and puts its counter back to zero.
// The heads of a pair are thus merged by up to four waves, usually on as many compute units, each behind its own
// stores only.  Nothing waits on another workgroup, and no cache is written back or invalidated as a whole (a
// device-scope fence costs tens of microseconds here).
// Measured against the previous form (a combine of two barriers, the whole workgroup's acknowledgement and count, one
// workgroup merging): 131072 rows, 8 KV heads, budget 4096: 10.9 -> 9.6 us; 4 x 32768 rows, budget 2048: 11.6 -> 11.1 us;
// 4096 rows, 2 KV heads, budget 256: 6.8 -> 6.4 us.
// red: G x 128 floats of LDS per wave, wave_stride floats apart.
// LOCAL (fast_cell): the pair's workgroups are dealt to one XCD, and the records stay in its L2: the acknowledgement and the
// record loads take a trip to the L2 instead of one to memory.  That the workgroups did meet on one XCD is not assumed:
// the counter, which stays at device scope, adds up their XCDs x and x^2 beside their number n, and n sum x^2 = (sum x)^2
// holds only if all x are the same.  If it does not, the records cannot be read; the function returns true, and the wave does
// the pair's whole list again for its heads.  That is no path to be on (4 x 32768 rows 10.1 -> 146 us a layer, 131072 8.6 -> 271: one
// wave, tile by tile): it is there for a dealing of workgroups other than round robin, which has not been seen.  Device scope / LOCAL, us a layer: 4096 rows, 2 KV heads 5.54 / 5.25; 4 x 32768 rows, 8 KV
// heads, budget 2048 10.55 / 10.28; 131072 rows, 8 KV heads, budget 4096 9.03 / 8.63; 8 sequences of 20011..24571 rows, G = 5, paged, budget 1024
// 12.29 / 11.85; 12 x 32768 rows, budget 1000 14.55 / 13.68; 8 x 32768 rows, one KV head, budget 2000 9.03 / 8.34.  (With the counter in the L2 as
// well another 1 %, but then workgroups on different XCDs would not find one another.)
// JSTAT (dense kernel with exposed logits): the record's header also carries the statistics over the allowed set J alone,
// { m, l, m_J, l_J } (the fast step and the dense kernel without logits leave the last two words).  2: m_J and l_J also go out for
// the pair's other workgroups, l_J with its sign bit set, so that they cannot be zero (score_tail).
// AT_ONCE: heads a wave merges at a time.  Two where a group has more than eight heads (the kernels with the plain K layout),
// so that up to four heads take two chains of trips, not four: 16 heads, 33 records, fast step 13.5 -> 12.8 us.  One for
// smaller groups, whose waves have one or two: the second head's code costs them 0.1 us.
template <int JSTAT = 0, int AT_ONCE = 1, bool LOCAL = false>
__device__ __forceinline__ bool finish_wg(const WgOut& o, int64_t head0, int G, int slot, const f32x4 (&acc)[8], float m_run,
                                          float l_run, float* red, int wave_stride, float m_j = 0.f, float l_j = 0.f) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jg = lane >> 4, n = lane & 15;
  __shared__ float s_m[16][kWaves];
  __shared__ float s_l[16][kWaves];
  __shared__ float s_mj[JSTAT ? 16 : 1][kWaves];
  __shared__ float s_lj[JSTAT ? 16 : 1][kWaves];
  if (lane < 16) {
    s_m[lane][w] = m_run;
    s_l[lane][w] = l_run;
    if (JSTAT) {
      s_mj[lane][w] = m_j;
      s_lj[lane][w] = l_j;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int hh = 4 * jg + i;
    if (hh < G) {
      float* dst = red + w * wave_stride + hh * kHeadDim + n * 8;
      *reinterpret_cast<float4*>(dst) = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
      *reinterpret_cast<float4*>(dst + 4) = make_float4(acc[4][i], acc[5][i], acc[6][i], acc[7][i]);
    }
  }
  __syncthreads();
  if (w >= G) return false;
  const int half = lane >> 5, c = lane & 31;
  constexpr int kRec = kPartStride * (int)sizeof(float);
  // slot_cap: records each query head has room for (kSlotCap in a caller's workspace, fewer in the static scratch)
  float* const pair_base = o.part + head0 * o.slot_cap * kPartStride;
  const __amdgpu_buffer_rsrc_t R = pair_records(pair_base, G * o.slot_cap * kRec);
  for (int h0 = w; h0 < G; h0 += 8) {
    const int hh = min(h0 + 4 * half, G - 1);
    const bool mine = h0 + 4 * half < G;
    const float4 m4 = *reinterpret_cast<const float4*>(&s_m[hh][0]), l4 = *reinterpret_cast<const float4*>(&s_l[hh][0]);
    float4 r[kWaves];
#pragma unroll
    for (int ww = 0; ww < kWaves; ++ww)
      r[ww] = *reinterpret_cast<const float4*>(red + ww * wave_stride + hh * kHeadDim + 4 * c);
    const float M = fmaxf(fmaxf(m4.x, m4.y), fmaxf(m4.z, m4.w));
    const float f[kWaves] = {fast_exp2(m4.x - M), fast_exp2(m4.y - M), fast_exp2(m4.z - M), fast_exp2(m4.w - M)};
    float4 t = make_float4(r[0].x * f[0], r[0].y * f[0], r[0].z * f[0], r[0].w * f[0]);
#pragma unroll
    for (int ww = 1; ww < kWaves; ++ww) {
      t.x += r[ww].x * f[ww]; t.y += r[ww].y * f[ww]; t.z += r[ww].z * f[ww]; t.w += r[ww].w * f[ww];
    }
    const float ls = l4.x * f[0] + l4.y * f[1] + l4.z * f[2] + l4.w * f[3];
    if (!JSTAT && o.out_direct != nullptr) {  // workgroup-uniform
      const float inv = ls > 0.f ? 1.0f / ls : 0.f;
      if (mine) store_out4(o.out_direct, (head0 + hh) * kHeadDim + 4 * c, make_float4(t.x * inv, t.y * inv, t.z * inv, t.w * inv), o.out_bf16);
    } else if (mine) {
      const int off = (hh * o.slot_cap + slot) * kRec;  // from the pair's first record
      if (!JSTAT && o.out_merge != nullptr) {
        store_record4<LOCAL>(R, off + 16 + 16 * c, t);
        if (c == 0) store_record2<LOCAL>(R, off, M, ls);
      } else {
        float* dst = pair_base + (hh * o.slot_cap + slot) * kPartStride;
        *reinterpret_cast<float4*>(dst + 4 + 4 * c) = t;
        if (JSTAT) {
          const float4 mj = *reinterpret_cast<const float4*>(&s_mj[hh][0]), lj = *reinterpret_cast<const float4*>(&s_lj[hh][0]);
          const float MJ = fmaxf(fmaxf(mj.x, mj.y), fmaxf(mj.z, mj.w));
          const float LJ = lj.x * fast_exp2(mj.x - MJ) + lj.y * fast_exp2(mj.y - MJ) + lj.z * fast_exp2(mj.z - MJ) + lj.w * fast_exp2(mj.w - MJ);
          if (JSTAT == 2 && c == 0)
            __hip_atomic_store(o.met + hh * kSlotCap + slot, (uint64_t)(__float_as_uint(LJ) | 0x80000000u) << 32 | __float_as_uint(MJ), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (c == 0) *reinterpret_cast<float4*>(dst) = make_float4(M, ls, MJ, LJ);
        } else if (c == 0) {
          *reinterpret_cast<float2*>(dst) = make_float2(M, ls);
        }
      }
    }
  }
  if (JSTAT || o.out_merge == nullptr) return false;
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's record stores have been performed
  const uint32_t xcd = LOCAL ? __builtin_amdgcn_s_getreg(20 | 3 << 11) : 0u;  // HW_REG_XCC_ID, 4 bits
  const uint32_t mine = 1u | xcd << 7 | (xcd * xcd) << 17;  // (at most 63 workgroups, XCDs 0 .. 15: no field overflows)
  uint32_t before = 0;
  if (lane == 0) before = __hip_atomic_fetch_add(o.arrive + w * kArriveStride, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint32_t total = (uint32_t)__builtin_amdgcn_readfirstlane((int)before) + mine;
  if ((total & 127u) != (uint32_t)o.n_split) return false;
  if (lane == 0) __hip_atomic_store(o.arrive + w * kArriveStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (LOCAL) {
    const uint32_t sum = (total >> 7) & 1023u, squares = total >> 17;
    if (__builtin_expect((uint32_t)o.n_split * squares != sum * sum, 0)) return true;
  }
  const int n_rec = o.n_split;
  for (int hh = w; hh < G; hh += AT_ONCE * kWaves) {
    const bool two = AT_ONCE > 1 && hh + kWaves < G;  // wave-uniform
    int P[AT_ONCE];  // byte offsets of the heads' records
    float M[AT_ONCE], Z[AT_ONCE];
    float4 t[AT_ONCE];
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) {
      P[k] = (hh + k * kWaves) * o.slot_cap * kRec;
      M[k] = kNeg;
      Z[k] = 0.f;
      t[k] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    for (int s0 = half; s0 - half < n_rec; s0 += 16) {  // this half's records s0, s0 + 2, ...
      float2 ml[AT_ONCE][8];
      float4 r4[AT_ONCE][8];
#pragma unroll
      for (int k = 0; k < AT_ONCE; ++k) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int rec = P[k] + min(s0 + 2 * i, n_rec - 1) * kRec;
          if ((k == 0 || two) && (i == 0 || s0 - half + 2 * i < n_rec)) {  // wave-uniform
            ml[k][i] = load_record2<LOCAL>(R, rec);
            r4[k][i] = load_record4<LOCAL>(R, rec + 16 + 16 * c);
          } else {
            ml[k][i] = make_float2(kNeg, 0.f);
            r4[k][i] = make_float4(0.f, 0.f, 0.f, 0.f);
          }
        }
      }
#pragma unroll
      for (int k = 0; k < AT_ONCE; ++k) {
        if (k > 0 && !two) break;
        float Mn = M[k];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          if (s0 + 2 * i >= n_rec) ml[k][i] = make_float2(kNeg, 0.f);
          Mn = fmaxf(Mn, ml[k][i].x);
        }
        const float f = fast_exp2(M[k] - Mn);
        Z[k] *= f;
        t[k].x *= f; t[k].y *= f; t[k].z *= f; t[k].w *= f;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const float wgt = fast_exp2(ml[k][i].x - Mn);
          const float wl = s0 + 2 * i < n_rec ? wgt : 0.f;  // (a half without any record has Mn = kNeg and weights 1)
          Z[k] += wl * ml[k][i].y;
          t[k].x += wl * r4[k][i].x; t[k].y += wl * r4[k][i].y; t[k].z += wl * r4[k][i].z; t[k].w += wl * r4[k][i].w;
        }
        M[k] = Mn;
      }
    }
#pragma unroll
    for (int k = 0; k < AT_ONCE; ++k) {
      if (k > 0 && !two) break;
      // the two halves' sums meet
      const float Mo = half_max(M[k]);
      const float f = fast_exp2(M[k] - Mo);
      const float Zs = half_sum(Z[k] * f);
      const float4 ts = make_float4(half_sum(t[k].x * f), half_sum(t[k].y * f), half_sum(t[k].z * f), half_sum(t[k].w * f));
      const float inv = Zs > 0.f ? 1.0f / Zs : 0.f;
      if (half == 0)
        store_out4(o.out_merge, (head0 + hh + k * kWaves) * kHeadDim + 4 * c, make_float4(ts.x * inv, ts.y * inv, ts.z * inv, ts.w * inv), o.out_bf16);
    }
  }
  return false;
}
// LOCAL, records that cannot be read: the wave has the whole list's sums and writes its heads w, w + 4, ... itself.
__device__ __forceinline__ void store_heads(const WgOut& o, int64_t head0, int G, const f32x4 (&acc)[8], float l_run) {
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jg = lane >> 4, n = lane & 15;
  const float l_n = rows_sum(l_run);  // of head n
  const float l4[4] = {row_quad<0>(l_n), row_quad<1>(l_n), row_quad<2>(l_n), row_quad<3>(l_n)};
  float l = 0.f, v[8];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (i != w) continue;
    l = l4[i];
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = acc[e][i];
  }
  const float inv = l > 0.f ? 1.0f / l : 0.f;
  if (4 * jg + w < G) {
    const int64_t at = (head0 + 4 * jg + w) * kHeadDim + 8 * n;
    store_out4(o.out_merge, at, make_float4(v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv), o.out_bf16);
    store_out4(o.out_merge, at + 4, make_float4(v[4] * inv, v[5] * inv, v[6] * inv, v[7] * inv), o.out_bf16);
  }
}

// Walks a position list whose rows are not consecutive: sink ++ sel ++ recent (gather), or
// sink ++ recent (the dense kernel's last workgroup, n_sel = 0).  Position p < nS is row p, then
// nSel selected rows, then rows rs, rs + 1, ...; positions past the list read row 0 with weight 0.
struct ListWalk {
  const int32_t* sel;  // row of sel_idx of this (b, h), or nullptr
  int sel_cap;         // sel_stride - 1
  int n_sink;
  int nS, nSel, rs, N;
  int r_hi;            // last readable row, max(L, 1) - 1: a stored index outside [0, r_hi] reads as r_hi
  int bad;
  __device__ __forceinline__ void set_counts(int L, int n_sel, int recent_start, int sel_stride) {
    nS = min(n_sink, L);
    nSel = min(max(n_sel, 0), sel_stride);
    bad |= nSel != n_sel ? kGuardNSel : 0;
    rs = min(max(recent_start, nS), L);
    N = nS + nSel + (L - rs);
    r_hi = max(L, 1) - 1;
  }
  __device__ __forceinline__ int sel_at_nonempty(int p) const {  // index stored for list position p (valid inside the sel part)
    return sel[min(max(p - n_sink, 0), sel_cap)];
  }
  __device__ __forceinline__ int row_of(int p, int s) {
    const int i = p - nS;
    int r = i < nSel ? s : rs + (i - nSel);
    r = p < nS ? p : r;
    r = p < N ? r : 0;
    // Sink and recent rows are inside the context by construction, so only a stored index can change here.
    // One clamp for both ends: a negative row reads as a huge one.
    const int rc = (int)min((uint32_t)r, (uint32_t)r_hi);
    bad |= rc != r ? kGuardSelIdx : 0;
    return rc;
  }
};

// ------------------------------------------------------------------------------------------------
// dense kernel
// ------------------------------------------------------------------------------------------------
// PAGED: K / V are block pools addressed through the sequence's block table.
// EXPOSE 1: also write y over J for the Selector; 2: y and the squared key norms; 3, 4: y (and the norms) stay in LDS as far as they fit, for score_tail.
// BIG: twice the logits stash per wave, which leaves room for one workgroup per compute unit only
// (launches where every sequence is dense, and the planned launch, run one per unit anyway; the ragged
// step's launch with a workgroup per cell keeps two, although that kernel spills 6 to 26 of its 256 registers: with one,
// 12 sequences of 5003 to 30011 rows, 4 of them slow, take 110 us a step instead of 104, 1100 of 100 to 500 rows, 100 slow,
// 249 instead of 215).
// PLANNED: the caller has the sequence's length and a range of its tiles (attn_dense_planned_kernel).
struct DenseShare {
  int first, step;   // tiles of wave w: first + w, first + w + step, ... below end (step: a multiple of the waves)
  int end;
  int slot, n_rec;   // the workgroup's record among the pair's
  int L, recent;     // PLANNED: rows the query sees, and what of the recent window it sees
  int bad;           // PLANNED: guard bits so far
  bool have_k;       // PLANNED: K rows of the first tile are on their way into T
};
// Floats of lds per wave: the logits stash, and at the end the wave's O for the combine (finish_wg).  EXPOSE 3: the four waves' O in
// front, then their stashes, which outlive it (score_tail), then the list of the sequences the workgroup has had.
constexpr int kScoreEntryFloats = 8;
constexpr int patch_floats(int expose, bool big) {
  return expose >= 3 ? (kScoreFloats + kScoreCap * kScoreEntryFloats) / kWaves : expose == 0 ? 16 * kHeadDim : big ? 2 * kStashFloats : kStashFloats;
}
struct Scored {
  int4* entry;  // two words per sequence: { head, sequence, first, step }, { end of J's tiles, |J|, records, own record }
  int n;        // sequences so far
  int used;     // tiles of J this wave has had so far
};
__device__ __forceinline__ Scored scored_of(float* lds) { return Scored{reinterpret_cast<int4*>(lds + kScoreFloats), 0, 0}; }
template <int EXPOSE, bool PAGED, bool BIG, bool WIDE, bool PLANNED>
__device__ __forceinline__ void dense_body(const AttnArgs& a, const DenseShare& sh, const int h, const int b, Tile& T, float* lds, Scored& sc, const int tid_bias = 0) {
  constexpr int kStash = BIG ? 2 * kStashFloats : kStashFloats;
  constexpr int kPatch = patch_floats(EXPOSE, BIG);
  constexpr bool SCORE = EXPOSE >= 3, NORM = EXPOSE == 2 || EXPOSE == 4;
  // everything uniform is asked for at once (the first argument load of a wave takes 0.4 us)
  asm volatile("" ::"s"(a.q), "s"(a.K), "s"(a.V), "s"(a.k_sb), "s"(a.k_sh), "s"(a.k_st), "s"(a.v_sb), "s"(a.v_sh), "s"(a.v_st),
               "s"(a.ctx_len), "s"(a.is_slow), "s"(a.q_len), "s"(a.Hq), "s"(a.Hkv), "s"(a.G), "s"(a.n_sink), "s"(a.recent),
               "s"(a.max_tiles), "s"(a.row_cap), "s"(a.len_cap));
  // the length is on its way before the first rows: behind them it would take the loaded memory's 1.5 us
  const int L_in = PLANNED ? 0 : a.ctx_len[b * a.ms];
  if (!PLANNED && a.is_slow != nullptr && a.is_slow[b * a.fs] == 0) return;
  const int tid = threadIdx.x + tid_bias;  // (tid_bias: zero; see attn_dense_planned_kernel)
  const int lane = tid & 63, w = tid >> 6;
  const int jg = lane >> 4, n = lane & 15;
  const int G = a.G;
  const int bh = b * a.Hkv + h;
  const int64_t head0 = (int64_t)b * a.Hq + h * G;
  Rows R;
  R.Kb = reinterpret_cast<const char*>(a.K + b * a.k_sb + h * a.k_sh);
  R.Vb = reinterpret_cast<const char*>(a.V + b * a.v_sb + h * a.v_sh);
  R.k_st = (uint32_t)a.k_st * 2u;
  R.v_st = (uint32_t)a.v_st * 2u;
  R.k_lane = k_lane_of<WIDE>(jg, n);
  R.v_lane = n * 16;
  R.jg = jg;
  R.n = n;

  // The prefix of (b, h) is cut into 32-row tiles in two runs: tiles [0, nTJ) cover the allowed set J
  // (tile t, position i is cache row n_sink + 32 t + i), tiles [nTJ, nTJ + nTS) cover the sink rows
  // followed by the recent window, which the Selector never ranks.  The waves of the workgroups on a
  // (b, h) pair share its tiles evenly.  A wave's J tiles come first: the J-only softmax statistics the Selector needs
  // are the wave's running ones at the point where its J tiles end.
  // Not PLANNED, the rows of the wave's first tile follow from the block index alone (almost always a J tile):
  // their loads go out before ctx_len arrives, clamped to the launch's row bound.
  const int first = sh.first + w, step = sh.step;
  // (a paged cache has valid blocks only up to ctx_len: no load before ctx_len is known)
  if (!PLANNED && !PAGED && first < a.max_tiles) {
    issue_k_affine<WIDE>(T, R, a.n_sink + first * kTile, a.row_cap);
    issue_v_affine<WIDE>(T, R, a.n_sink + first * kTile, a.row_cap);
  }
  bf16x8 qreg[4];
  load_q_raw<WIDE>(qreg, a.q, head0, G, jg, n);
  int bad = PLANNED ? sh.bad : 0;
  int L = sh.L, recent = sh.recent;  // a window query under the causal mask sees a shorter context with what is left of the recent window
  if (!PLANNED) window_view(a.q_len, b, guarded_len(L_in, a.len_cap, bad), a.recent, L, recent);
  const int NJ = max(0, L - recent - a.n_sink);
  const int nTJ = (NJ + kTile - 1) / kTile;
  const int rJ_max = a.n_sink + NJ - 1;
  const int nS = min(a.n_sink, L);
  const int rs = min(max(a.n_sink, L - recent), L);
  const int NS = nS + (L - rs);
  const int nTS = (NS + kTile - 1) / kTile;
  const int nT = PLANNED ? min(sh.end, nTJ + nTS) : nTJ + nTS;
  const int nTJw = min(nTJ, nT);
  const int K = first < nT ? (nT - first + step - 1) / step : 0;      // tiles of this wave
  const int KJ = first < nTJw ? (nTJw - first + step - 1) / step : 0;  // ... of which in J
  const int d_rs = rs - nS, r_last = max(L, 1) - 1;
  // cache row of position i of tile t; tiles past the end (the refill after the last tile) read row L - 1
  // (row 0 of an empty context: the cache holds max_ctx >= 1 rows)
  auto row_for = [&](int t, int i) -> int {
    const int xj = a.n_sink + t * kTile + i;
    const int xs = (t - nTJ) * kTile + i;
    const int r_s = min(xs < nS ? xs : xs + d_rs, r_last);
    return t < nTJ ? min(xj, rJ_max) : r_s;
  };
  auto issue_k_tile = [&](Tile& T, int t) {
    if (WIDE) {  // whole 128-byte lines: position 8 * blk + (n & 7), the half of the row this lane's column belongs to
#pragma unroll
      for (int blk = 0; blk < 4; ++blk) {
        const uint32_t o = (uint32_t)row_for(t, 8 * blk + (n & 7)) * R.k_st + R.k_lane;
        wide_k(T, blk, 0) = load_row16(R.Kb, o);
        wide_k(T, blk, 1) = load_row16(R.Kb, o, 128);
      }
      return;
    }
    const uint32_t oa = (uint32_t)row_for(t, n) * R.k_st + R.k_lane;
    const uint32_t ob = (uint32_t)row_for(t, 16 + n) * R.k_st + R.k_lane;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      T.ka[kb] = load_row16(R.Kb, oa, kb * 64);
      T.kb[kb] = load_row16(R.Kb, ob, kb * 64);
    }
  };
  auto issue_v_tile = [&](Tile& T, int t) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      T.v[i] = load_row16(R.Vb, (uint32_t)row_for(t, slot_pos<WIDE>(jg, i)) * R.v_st + R.v_lane);
      T.v[4 + i] = load_row16(R.Vb, (uint32_t)row_for(t, slot_pos<WIDE>(jg, 4 + i)) * R.v_st + R.v_lane);
    }
  };
  Pages P;
  int pra2 = 0, prb2 = 0;  // PAGED: physical rows of the second tile
  int pa_n = 0, pb_n = 0;  // PAGED: block-table entries of the next refill's K rows (this lane's rows n and 16 + n)
  if (PAGED) {
    // Same order of memory instructions as an iteration of the loop: K rows, the table entries of the next refill, V rows.
    // Waves without tiles read row L - 1.
    P = pages_of(a, b, L);
    const int ra = row_for(first, n), rb = row_for(first, 16 + n);
    const int ra2 = row_for(first + step, n), rb2 = row_for(first + step, 16 + n);
    const int pa = P.page_of(ra), pb = P.page_of(rb), pa2 = P.page_of(ra2), pb2 = P.page_of(rb2);
    const int pra = P.phys(ra, pa, bad), prb = P.phys(rb, pb, bad);
    pra2 = P.phys(ra2, pa2, bad);
    prb2 = P.phys(rb2, pb2, bad);
    __builtin_amdgcn_sched_barrier(0);
    issue_k_rows<uint64_t>(T, R, pra, prb);
    __builtin_amdgcn_sched_barrier(0);
    pa_n = P.page_of(row_for(first + 2 * step, n));
    pb_n = P.page_of(row_for(first + 2 * step, 16 + n));
    __builtin_amdgcn_sched_barrier(0);
    issue_v_rows<uint64_t>(T, R, pra, prb);
    __builtin_amdgcn_sched_barrier(0);
  } else if (K > 0 && (PLANNED || first >= nTJ)) {  // (short context: the first tile is a sink / recent tile after all)
    if (!PLANNED || !sh.have_k || first >= nTJ) issue_k_tile(T, first);
    issue_v_tile(T, first);
  }
  // Two tiles are in flight per wave: the second buffer takes the wave's second tile now.
  Tile T2;
  constexpr int NB = 2;  // tile buffers; a tile's refill is the wave's tile NB further on
  if (K > 1) {
    __builtin_amdgcn_sched_barrier(0);
    if (PAGED) {
      issue_k_rows<uint64_t>(T2, R, pra2, prb2);
      issue_v_rows<uint64_t>(T2, R, pra2, prb2);
    } else {
      issue_k_tile(T2, first + step);
      issue_v_tile(T2, first + step);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  mask_q<WIDE>(qreg, G, n);

  float m_run = kNeg, l_run = 0.f;
  float m_j = kNeg, l_j = 0.f;  // the same over J alone
  f32x4 acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Exposing y.  The logits of (b, h) are stored tile-major, [tile][G heads][32 positions], so a
  // tile's G x 128 bytes are one contiguous run.  A wave does not store a tile's logits when it
  // has them: a store acknowledged late would sit in front of the next rows in the in-order
  // memory counter.  It parks them in its LDS stash, laid out as they go to memory, and writes the
  // stash out in one burst when it is full and once more after its last tile, when nothing is
  // left to wait for.
  // With NORM a tile has one more row: ||k_j||^2 of its 32 positions, for the key-norm factor of
  // the Selector's prior (Eq. selector_prior_kn).
  const int rows_exp = G + (NORM ? 1 : 0);
  float* stash = SCORE ? lds + kWaves * G * kHeadDim + w * score_stash_floats(G) : lds + w * kPatch;
  float* lg_base = EXPOSE != 0 ? a.logits + (int64_t)bh * rows_exp * a.ld_pos : nullptr;
  const int tile_f4 = rows_exp * (kTile / 4);        // float4 per tile
  // EXPOSE 3: the first tiles stay where they are, for score_tail; what goes to memory lies behind them.
  const int stay = SCORE ? score_stay(G, rows_exp) : 0;
  const int stash_cap = SCORE ? kScoreBurst : kStash / (rows_exp * kTile);  // tiles the stash holds until they are written
  int n_stashed = 0, k_flushed = SCORE ? max(0, stay - sc.used) : 0;
  const float* const burst = stash + stay * (rows_exp * kTile);
  auto flush_stash = [&]() {
    __builtin_amdgcn_wave_barrier();
    const int n_f4 = n_stashed * tile_f4;
    for (int f = lane; f < n_f4; f += 64) {
      const int i = f / tile_f4, rem = f - i * tile_f4;
      const int t = first + (k_flushed + i) * step;
      *reinterpret_cast<float4*>(lg_base + ((int64_t)t * tile_f4 + rem) * 4) = *reinterpret_cast<const float4*>(burst + f * 4);
    }
    __builtin_amdgcn_wave_barrier();
    k_flushed += n_stashed;
    n_stashed = 0;
  };
  // One loop for all of the wave's tiles.  A tile buffer's K half is refilled with the rows of the
  // tile that uses the buffer next as soon as the logits are out, its V half as soon as P V is done,
  // so rows are on their way during all of the math (with two buffers, a whole tile more than with
  // one).  No branch surrounds a load, so that every wait can name exactly the loads it needs; the last tiles have
  // copies of the body without the refill (the requests of a refill that reads nothing new cost a wave 0.2 us).
  auto tile_step = [&](Tile& T, int k, auto refill) {
    constexpr bool kRefill = decltype(refill)::value;
    const int t = first + k * step;
    const bool inJ = k < KJ;
    if (EXPOSE != 0 && k == KJ) {  // the J tiles are done (or there were none)
      m_j = m_run;
      l_j = l_run;
    }
    float y[8];
    f32x4 s4[4];
    if (WIDE) qk_products_wide(T, qreg, s4);  // the refill of the K half below goes out before the lane exchanges
    else qk_phase(T, qreg, a.scale_log2, y);
    float k2a = 0.f, k2b = 0.f;
    if (NORM) knorm_phase(T, jg, n, k2a, k2b);
    int pra = 0, prb = 0;
    if (!kRefill) {
    } else if (PAGED) {
      pra = P.phys(row_for(t + NB * step, n), pa_n, bad);
      prb = P.phys(row_for(t + NB * step, 16 + n), pb_n, bad);
      issue_k_rows<uint64_t>(T, R, pra, prb);
      pa_n = P.page_of(row_for(t + (NB + 1) * step, n));
      pb_n = P.page_of(row_for(t + (NB + 1) * step, 16 + n));
    } else {
      issue_k_tile(T, t + NB * step);
    }
    if (WIDE) {
      __builtin_amdgcn_sched_barrier(0);
      qk_join_wide(s4, a.scale_log2, y);
    }
    if (EXPOSE != 0 && inJ) {  // positions past |J| land in the padding of the last tile, never used
      const bool stays = SCORE && sc.used + k < stay;
      float* st = stash + (SCORE ? min(sc.used + k, stay) + n_stashed : n_stashed) * (rows_exp * kTile);
      stage_logits<WIDE>(st, y, jg, n, G);
      if (NORM && jg == (n >> 2)) {
        st[G * kTile + n] = k2a;
        st[G * kTile + 16 + n] = k2b;
      }
      if (!stays && ++n_stashed == stash_cap) flush_stash();
    }
    const int p0 = (inJ ? t : t - nTJ) * kTile;
    const int N = inJ ? NJ : NS;
    if (p0 + kTile > N) mask_tail<WIDE>(T, y, jg, p0, N);
    bf16x8 a_hi, a_lo;
    softmax_phase(y, acc, m_run, l_run, jg, a_hi, a_lo);
    pv_phase(T, a_hi, a_lo, acc);
    if (!kRefill) return;
    if (PAGED) issue_v_rows<uint64_t>(T, R, pra, prb);
    else issue_v_tile(T, t + NB * step);
  };
  const std::integral_constant<bool, true> refill;
  const std::integral_constant<bool, false> last;
  if (K == 1) {
    tile_step(T, 0, last);
  } else if (K > 1) {
    // (an odd last tile is taken after the loop: a way out of the middle of the loop body would put a
    // path from the first buffer's refill straight to its next use into the flow graph, and the waits
    // would be placed for that path)
    int k = 0;
    for (; k + 2 < K; k += 2) {
      tile_step(T, k, refill);
      tile_step(T2, k + 1, refill);
    }
    if (k + 1 < K) {
      tile_step(T, k, last);
      tile_step(T2, k + 1, last);
    } else {
      tile_step(T, k, last);
    }
  }
  if (EXPOSE != 0) flush_stash();
  if (EXPOSE != 0 && K == KJ) {
    m_j = m_run;
    l_j = l_run;
  }
  WgOut o = wg_out_of(a, bh);
  o.n_split = sh.n_rec;
  if (SCORE) o.met = a.met + (int64_t)bh * G * kSlotCap;
  if (PLANNED && sh.n_rec == 1) {
    o.out_direct = o.out_merge;
    o.out_merge = nullptr;
  }
  finish_wg<SCORE ? 2 : EXPOSE != 0>(o, head0, G, sh.slot, acc, m_run, rows_sum(l_run), lds, SCORE ? G * kHeadDim : kPatch, m_j,
                                           EXPOSE != 0 ? rows_sum(l_j) : 0.f);
  if (SCORE) {
    sc.used += KJ;
    if (tid == 0) {
      sc.entry[2 * sc.n] = make_int4(h, b, sh.first, sh.step);
      sc.entry[2 * sc.n + 1] = make_int4(nTJw, NJ, sh.n_rec, sh.slot);
    }
    ++sc.n;
  }
  report_guard(a.guard, bad);
}
// ---- scoring in the dense launch (EXPOSE 3, 4) ------------------------------------------------------------------
// The evidence of a position is a sum over the group's heads, each over its own normaliser (Eq. selector_mu), and those are known
// when all workgroups of a pair have left their statistics.  A workgroup that has done its share therefore waits for
// the pair's others and turns the logits, which it still has in LDS, into keys and a histogram of its own: a G-th of the
// bytes to memory, and no scoring launch.
// A workgroup's statistics of a head are one word of eight bytes that is never zero, written and read at device scope and put back
// to zero by the Selector's last launch: what has arrived is seen in the value itself, so nothing is ordered or counted.  (A
// counter behind acknowledged headers, in front of their loads, was 0.7 us longer, in the L2 of one XCD no shorter.)
// All workgroups of the launch are on the chip together where it has the chip to itself (score_in_dense); where it has
// not, some may only start when others have ended, so the wait has a limit.  Behind it a workgroup writes its logits and leaves its
// record to the pair's others: it marks it in the pair's mask and counts itself out.  The others count themselves out when all they have is scored: who then
// finds that records of the pair were left claims them from the mask one by one, and the pair's last one, who
// finds the statistics complete whatever the others saw, takes all that nobody has claimed.  So every record is
// scored once, in this launch, and the next one does not see which way it went.  (With every record left, which the last workgroups of the pairs
// then work off alone, us a slow step of 4 x 32768 rows 103 -> 125, of 1 x 131071 with the full Selector 117 -> 288; left to the Selector's launches, of which each workgroup
// scored all of them again, 140 and 880.)  Counting at the end of each sequence instead, with the answer looked at behind its keys, made the way to the next
// one wait for them: 8 x 20011..24571 rows, G = 5, paged 135.3 -> 133.7 us for the present form.
// Nothing of this is decided before all of the workgroup's own shares are done and out, so no workgroup waits for one that waits.
// The keys are bit for bit what the scoring launch (sel_score_kernel) makes of the same logits.
// FULL: evidence, prior and their sums for the full Selector, as sel_prior_kernel leaves them (the sums per workgroup, not per segment).
// A record that was left is handed over without a fence: its logits and tiles go out and come back at device scope, and are performed before the mask
// has its bit.
__device__ __forceinline__ void store_far4(float* dst, float4 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(dst), (uint64_t)__float_as_uint(v.y) << 32 | __float_as_uint(v.x), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(reinterpret_cast<uint64_t*>(dst) + 1, (uint64_t)__float_as_uint(v.w) << 32 | __float_as_uint(v.z), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float4 load_far4(const float* src) {
  const uint64_t a = __hip_atomic_load(reinterpret_cast<const uint64_t*>(src), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const uint64_t b = __hip_atomic_load(reinterpret_cast<const uint64_t*>(src) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float4(__uint_as_float((uint32_t)a), __uint_as_float((uint32_t)(a >> 32)), __uint_as_float((uint32_t)b), __uint_as_float((uint32_t)(b >> 32)));
}
// Records of the mask that are this workgroup's from now on: all there are, or one (0: there is none).
__device__ __forceinline__ uint64_t claim_left(unsigned long long* mask, bool every) {
  if (every) return __hip_atomic_exchange(mask, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint64_t m = __hip_atomic_load(mask, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  while (m != 0) {  // (at most one trip per record: a bit that somebody else has claimed does not come back)
    const uint64_t bit = m & (0 - m);
    const uint64_t old = __hip_atomic_fetch_and(mask, ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((old & bit) != 0) return bit;
    m = old & ~bit;
  }
  return 0;
}
// An entry of the workgroup's list, in scalar registers.
struct ScoredEntry {
  int h, b, first, step, end, NJ, n_rec, slot;
};
__device__ __forceinline__ ScoredEntry scored_entry(const Scored& sc, int e) {
  const int4 e0 = sc.entry[2 * e], e1 = sc.entry[2 * e + 1];
  return ScoredEntry{__builtin_amdgcn_readfirstlane(e0.x), __builtin_amdgcn_readfirstlane(e0.y), __builtin_amdgcn_readfirstlane(e0.z),
                     __builtin_amdgcn_readfirstlane(e0.w), __builtin_amdgcn_readfirstlane(e1.x), __builtin_amdgcn_readfirstlane(e1.y),
                     __builtin_amdgcn_readfirstlane(e1.z), __builtin_amdgcn_readfirstlane(e1.w)};
}
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
template <bool FULL>
__device__ __forceinline__ void score_tail(const AttnArgs& a, const Scored& sc, float* lds) {
  __shared__ __align__(16) uint32_t s_hist[FULL ? 2 * kAttnThreads : kHistBins];
  __shared__ double s_sums[kWaves][kSegStats];
  __shared__ float s_M[16], s_c[16];
  __shared__ uint32_t s_met[kWaves];
  __shared__ uint8_t s_out[kScoreCap];  // of an entry: OUT_...
  __shared__ uint64_t s_mask[2];
  __shared__ int4 s_tiles[kSlotCap];  // of the records claimed
  enum { OUT_SCORED = 0, OUT_LEFT = 1, OUT_LAST = 2 };  // scored and not counted out yet; left; left, and the pair's last one
  static_assert(kHistBins == 2 * kAttnThreads, "two bins, or one word of a segment's histogram, per thread");
  static_assert(kScoreCap <= 64 && kSlotCap <= 64, "an entry, a record per lane");
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.G, rows = G + (FULL ? 1 : 0), tile_f = rows * kTile, stay = score_stay(G, rows);
  const float* const stash = lds + kWaves * G * kHeadDim + w * score_stash_floats(G);
  reinterpret_cast<uint2*>(s_hist)[tid] = make_uint2(0u, 0u);
  __syncthreads();  // (the list is there)
  const uint64_t t0 = wall_clock64();  // the limit is for all sequences together
  const uint64_t limit = (uint64_t)abs(a.met_ticks);
  auto tiles_of_wave = [&](int first, int step, int end) { return first < end ? (end - first + step - 1) / step : 0; };
  // The statistics of a pair's heads, to s_M and s_c: wave w takes heads w, w + 4, ..., a record per lane.  WAIT: until they are there or the limit is over
  // (false: they are not); else they are known to be.
  auto statistics = [&](const ScoredEntry& E, int bh, auto WAIT) -> bool {
    bool all = true;
    for (int g = w; g < 16; g += kWaves) {
      float M = -kNeg, c = 0.f;  // (heads past the group count for nothing)
      if (g < G) {
        const uint64_t* const met = a.met + ((int64_t)bh * G + g) * kSlotCap + min(lane, E.n_rec - 1);
        uint64_t v = 0;
        if (WAIT) {
          all = false;
          while (limit > 0) {
            v = __hip_atomic_load(met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            all = __all(v != 0 && a.met_ticks > 0);
            if (all || wall_clock64() - t0 >= limit) break;
            __builtin_amdgcn_s_sleep(2);
          }
          if (!all) break;
        } else {
          v = __hip_atomic_load(met, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        const float2 ml = lane < E.n_rec ? make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32) & 0x7fffffffu)) : make_float2(kNeg, 0.f);
        c = group_stat(ml, a.alpha, G, M);
      }
      if (lane == 0) {
        s_M[g] = M;
        s_c[g] = c;
      }
    }
    return all;
  };
  double sums[kSegStats];
  // (FULL: this wave's sums, of one record, in front of the barrier behind which they are stored)
  auto put_sums = [&]() {
    if (!FULL) return;
#pragma unroll
    for (int i = 0; i < kSegStats; ++i) sums[i] = wave_sum_d(sums[i]);
    if (lane == 0) {
#pragma unroll
      for (int i = 0; i < kSegStats; ++i) s_sums[w][i] = sums[i];
    }
  };
  int used = 0;  // tiles of this wave in front of the sequence's
  for (int e = 0; e < sc.n; ++e) {
    const ScoredEntry E = scored_entry(sc, e);
    const int first = E.first + w, KJ = tiles_of_wave(first, E.step, E.end), in_lds = max(0, min(KJ, stay - used));
    const int bh = E.b * a.Hkv + E.h;
    const float* const kept = stash + used * tile_f;
    float* const lg = a.logits + (int64_t)bh * tile_f / kTile * a.ld_pos;
    used += KJ;
    if (in_lds < KJ) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the wave's other logits are written
    if (FULL)  // (the next launch adds to the segments' histograms)
      for (int sg = E.slot; sg * kSelSeg < E.NJ; sg += E.n_rec) a.hist[((int64_t)bh * a.n_seg_cap + sg) * (kHistBins / 2) + tid] = 0u;
    const bool all = statistics(E, bh, std::true_type{});
    if (lane == 0) s_met[w] = all;
    __syncthreads();
    if ((s_met[0] & s_met[1] & s_met[2] & s_met[3]) == 0u) {  // workgroup-uniform: the record is left
      for (int f = lane; f < KJ * (tile_f / 4); f += 64) {  // (logits beyond LDS are in memory already, but perhaps only in this XCD's L2)
        const int i = f / (tile_f / 4), rem = f - i * (tile_f / 4);
        float* const dst = lg + (int64_t)(first + i * E.step) * tile_f + rem * 4;
        if (i < in_lds) store_far4(dst, *reinterpret_cast<const float4*>(kept + f * 4));
        else store_far4(dst, *reinterpret_cast<const float4*>(dst));
      }
      if (tid == 0) {
        uint64_t* const tiles = reinterpret_cast<uint64_t*>(a.met_tiles + (int64_t)bh * kSlotCap + E.slot);
        __hip_atomic_store(tiles, (uint64_t)(uint32_t)E.step << 32 | (uint32_t)E.first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(tiles + 1, (uint64_t)(uint32_t)E.end, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's statistics, logits and tiles have been performed
      __syncthreads();
      if (tid == 0) {
        const uint64_t was = __hip_atomic_fetch_or(a.met_out + 2 * bh, 1ull << E.slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::"v"((uint32_t)was) : "memory");  // (in the mask before it is counted)
        const uint64_t out = __hip_atomic_fetch_add(a.met_out + 2 * bh + 1, 1ull << 32 | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_out[e] = (uint32_t)out == (uint32_t)(E.n_rec - 1) ? OUT_LAST : OUT_LEFT;
      }
      continue;  // (s_met is written again by the other waves only when they have seen the barrier above)
    }
    if (tid == 0) s_out[e] = OUT_SCORED;
    const int64_t row = (int64_t)bh * a.ld_pos;
    const Prior prior(a.prior_args, E.NJ);
#pragma unroll
    for (int i = 0; i < kSegStats; ++i) sums[i] = 0.0;
    auto score = [&](int p, const float* src) {
      float f[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
      for (int g = 0; g < G; ++g) add_evidence(f, *reinterpret_cast<const float4*>(src + g * kTile), a.alpha, s_M[g], s_c[g]);
      rank_quad<FULL>(a, row, E.NJ, prior, sums, s_hist, p, f, FULL ? *reinterpret_cast<const float4*>(src + G * kTile) : make_float4(0.f, 0.f, 0.f, 0.f));
    };
    for (int k0 = 0; k0 < KJ; k0 += 8) {  // eight tiles at a time, a quad of positions per lane
      const int k = k0 + (lane >> 3), t = first + k * E.step, p = t * kTile + (lane & 7) * 4;
      if (p >= E.NJ) continue;
      if (k < in_lds) score(p, kept + k * tile_f + (lane & 7) * 4);
      else if (k < KJ) score(p, lg + (int64_t)t * tile_f + (lane & 7) * 4);
    }
    put_sums();
    __syncthreads();
    store_record_stats<FULL>(a, (int64_t)bh * kSlotCap + E.slot, s_hist, s_sums);  // (the next record is scored behind a barrier)
  }
  // Out: an entry per lane.
  __syncthreads();
  if (w == 0) {
    uint64_t help = 0, last = 0;
    if (lane < sc.n) {
      const int4 e0 = sc.entry[2 * lane], e1 = sc.entry[2 * lane + 1];
      const int how = s_out[lane];
      uint64_t out = 0;
      if (how == OUT_SCORED) out = __hip_atomic_fetch_add(a.met_out + 2 * (e0.y * a.Hkv + e0.x) + 1, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = how == OUT_LAST || (how == OUT_SCORED && (uint32_t)out == (uint32_t)(e1.z - 1));
      help = how == OUT_LAST || out >> 32 != 0;
    }
    help = __ballot(help != 0);
    last = __ballot(last != 0);
    if (lane == 0) {
      s_mask[0] = help;
      s_mask[1] = last;
    }
  }
  __syncthreads();
  const uint64_t last = uniform64(s_mask[1]);
  for (uint64_t help = uniform64(s_mask[0]); help != 0; help &= help - 1) {
    const int e = __builtin_ctzll(help);
    const ScoredEntry E = scored_entry(sc, e);
    const int bh = E.b * a.Hkv + E.h;
    const float* const lg = a.logits + (int64_t)bh * tile_f / kTile * a.ld_pos;
    const int64_t row = (int64_t)bh * a.ld_pos;
    const Prior prior(a.prior_args, E.NJ);
    statistics(E, bh, std::false_type{});
    for (uint64_t claimed = 0;;) {
      __syncthreads();  // (statistics, histogram and sums of the record before)
      if (claimed == 0) {
        if (w == 0) {
          uint64_t m = 0;
          if (lane == 0) m = claim_left(a.met_out + 2 * bh, (last >> e & 1u) != 0);
          m = uniform64(m);
          if (m >> lane & 1u) {
            const uint64_t* const tiles = reinterpret_cast<const uint64_t*>(a.met_tiles + (int64_t)bh * kSlotCap + lane);
            const uint64_t x = __hip_atomic_load(tiles, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), y = __hip_atomic_load(tiles + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_tiles[lane] = make_int4((int)(uint32_t)x, (int)(x >> 32), (int)(uint32_t)y, 0);
          }
          if (lane == 0) s_mask[0] = m;
        }
        __syncthreads();
        claimed = uniform64(s_mask[0]);
        if (claimed == 0) break;
      }
      const int slot = __builtin_ctzll(claimed);
      claimed &= claimed - 1;
      const int4 tiles = s_tiles[slot];
      const int first = __builtin_amdgcn_readfirstlane(tiles.x) + w, step = __builtin_amdgcn_readfirstlane(tiles.y), K = tiles_of_wave(first, step, __builtin_amdgcn_readfirstlane(tiles.z));
#pragma unroll
      for (int i = 0; i < kSegStats; ++i) sums[i] = 0.0;
      for (int k0 = 0; k0 < K; k0 += 32) {  // the same lanes in the same order, four trips' requests at once
        float f[4][4] = {};
        const float* src[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) src[i] = lg + (int64_t)(first + min(k0 + 8 * i + (lane >> 3), K - 1) * step) * tile_f + (lane & 7) * 4;
#pragma unroll 4
        for (int g = 0; g < G; ++g) {
          float4 l[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) l[i] = load_far4(src[i] + g * kTile);
#pragma unroll
          for (int i = 0; i < 4; ++i) add_evidence(f[i], l[i], a.alpha, s_M[g], s_c[g]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int k = k0 + 8 * i + (lane >> 3);
          const float4 k2 = FULL ? load_far4(src[i] + G * kTile) : make_float4(0.f, 0.f, 0.f, 0.f);
          if (k < K) rank_quad<FULL>(a, row, E.NJ, prior, sums, s_hist, (first + k * step) * kTile + (lane & 7) * 4, f[i], k2);
        }
      }
      put_sums();
      __syncthreads();
      store_record_stats<FULL>(a, (int64_t)bh * kSlotCap + slot, s_hist, s_sums);
    }
  }
}
// One workgroup per (KV head, split, sequence) cell: wave w of split s takes tiles 4 s + w, 4 (s + n_split) + w, ...
// The head is the grid's first index here and in the planned launch, for the Selector's sake (Place in sfi_select.hip); by itself the order is worth
// nothing that could be told from noise (16 x 16384 rows, dense alone, splits first 157.9 us, heads first 157.2).
template <int EXPOSE, bool PAGED, bool BIG = false, bool WIDE = false>
__global__ __launch_bounds__(kAttnThreads, BIG ? 1 : 2) void attn_dense_kernel(const AttnArgs a) {
  const DenseShare sh{(int)blockIdx.y * kWaves, a.n_split * kWaves, 0, (int)blockIdx.y, a.n_split, 0, 0, 0, false};
  __shared__ __align__(16) float s_patch[kWaves * patch_floats(EXPOSE, BIG)];
  Tile T;
  Scored sc = scored_of(s_patch);
  dense_body<EXPOSE, PAGED, BIG, WIDE, false>(a, sh, blockIdx.x, blockIdx.z, T, s_patch, sc);
  if (EXPOSE >= 3) score_tail<EXPOSE == 4>(a, sc, s_patch);
}
// The launch planned on the device: more than one sequence, every one with a length of its own (which only the device
// knows) and, in the ragged step (sfi_mixed_step*), only some of them slow.  With a workgroup per cell the shares follow the
// sequences' lengths, and in the ragged step thousands of workgroups find nothing to do.  Here the tiles of the
// sequences taking part are laid end to end, per KV head, and cut into one equal share per workgroup (W per head, about
// one workgroup per compute unit in all), so that a workgroup's share can reach into several sequences; it leaves a
// record (and a combine) for each.
// - A position in the list counts in 1/1024 of a share; sequence r begins at X_r = P_r * scale + r (P_r: the tiles in
//   front of it), so that every sequence is at least 1 long.
// - A second sequence costs a workgroup its way out and its way in again, about kCross tiles' time: between two
//   sequences the list has kCross tiles of nothing.  A border that is closer to a share's end than half of that is moved
//   there instead, and then nothing is lost: sequences of equal lengths get whole workgroups.
// - The workgroups that have nothing but one sequence interleave their tiles (wave by wave, as in the launch above);
//   ranges of consecutive tiles would start at multiples of one large stride, and run at the same pace over the
//   same few memory channels.  The first and the last workgroup of a sequence take their part at its ends.
// - Every wave works out the plan by itself (a sequence per lane, a scan over the lanes; no LDS, no barrier), from
//   leading arguments that it has in registers when it starts.  The workgroup with a sequence's first record notes how many records it has, for the
//   launches that merge them, and the list of the sequences taking part for the Selector's.
struct PlanArgs {
  int W, n_on, total;
  float scale;
  int h;          // half a border's gap, in positions; also how far a border moves
  int n_a, s_b;   // CELLS: workgroups with a whole share of 1 << kShareLg positions, and the share of the others, which follow
};
constexpr int kShareLg = 10;
constexpr float kCross = 5.f;
// Where workgroup w's share begins, and whose share position x is in.
template <bool CELLS>
__device__ __forceinline__ int share_start(const PlanArgs& p, int w) {
  return !CELLS || w <= p.n_a ? w << kShareLg : (p.n_a << kShareLg) + (w - p.n_a) * p.s_b;
}
template <bool CELLS>
__device__ __forceinline__ int share_of(const PlanArgs& p, int x) {
  const int y = x - (p.n_a << kShareLg);
  if (!CELLS || y < 0) return x >> kShareLg;
  int w = (int)((float)y * __builtin_amdgcn_rcpf((float)p.s_b));
  w -= w * p.s_b > y;
  w += (w + 1) * p.s_b <= y;
  return p.n_a + w;
}
// Position of the border in front of sequence `rank` with P tiles before it; off: the gap on either side of it.
template <bool CELLS>
__device__ __forceinline__ int plan_border(const PlanArgs& p, int P, int rank, int& off) {
  int x = (int)((float)P * p.scale) + rank;
  const int w = share_of<CELLS>(p, x);
  const int f = x - share_start<CELLS>(p, w), up = share_start<CELLS>(p, w + 1) - x;
  const int h = CELLS && w >= p.n_a ? min(p.h, p.s_b >> 2) : p.h;
  off = f > h && up > h ? h : 0;
  x += f <= h ? -f : up <= h ? up : 0;
  if (P == 0) x = 0, off = 0;
  if (P == p.total) x = share_start<CELLS>(p, p.W), off = 0;
  return x;
}
// CELLS: the launch also has the ragged step's fast cells (attn_ragged_kernel), each as much work as `tiles` of this list's
// tiles.  Which workgroups have one follows from the flags; where there are enough without one, a workgroup that has had a cell
// takes that much less, so that all do the same in all.  There are then two sizes of shares, the whole ones first.  A
// sequence on both sides of the line between them is interleaved on each side by itself.  Where that
// takes less than kLeastGain tiles off the longest, the shares stay equal (32 x 8192 rows, one slow, 64.4 us a step, with two sizes 66.0; a
// line at 8 tiles: 16 x 16384..49152, 4 slow, 128.5 -> 132.9).
constexpr float kLeastGain = 4.f;
struct PlanCells {
  int n_split, row_lg;  // cells of a pair; log2 of the sequences whose cells alternate (fast_cell)
  float tiles;
  int L0, on0;          // length and flag of this lane's first sequence, requested in front of the cell's work
};
// GUESS: the workgroup requests its first rows on the guess that all sequences are equally long (a.plan_even).
template <int EXPOSE, bool PAGED, bool GUESS, bool CELLS = false>
__device__ __forceinline__ void planned_body(int j, int h, const int32_t* ctx_len, const uint8_t* is_slow, const int32_t* q_len,
                                             uint32_t strides, int B, int W_max, float per_min, int n_sink, int recent_in, int len_cap,
                                             const AttnArgs& a, float* lds, Scored& sc, const PlanCells cells = {}) {
  const int lane = threadIdx.x & 63;
  const int ms = strides & 0xffff, fs = strides >> 16;
  // rows seen, recent window seen and tiles of sequence b (at least one tile: an empty context has a record too)
  auto view_of = [&](int b, int L_in, int& L, int& recent, int& bad) -> int {
    window_view(q_len, b, guarded_len(L_in, len_cap, bad), recent_in, L, recent);
    const int NJ = max(0, L - recent - n_sink);
    const int nS = min(n_sink, L), rs = min(max(n_sink, L - recent), L);
    return max(1, (NJ + kTile - 1) / kTile + (nS + (L - rs) + kTile - 1) / kTile);
  };
  // this lane's sequences: per consecutive ones, tiles of sequence i among them (0: takes no part)
  const int per = (B + 63) / 64;
  auto tiles_of = [&](int b, int bc, int L_in, int on, int& L) -> int {
    int rec, bad = 0;
    const int t = view_of(bc, L_in, L, rec, bad);
    return b < B && on != 0 ? t : 0;
  };
  auto lane_seq = [&](int i, int& L_in, int& L) -> int {
    const int b = lane * per + i, bc = min(b, B - 1);
    L_in = ctx_len[bc * ms];
    return tiles_of(b, bc, L_in, is_slow == nullptr || is_slow[bc * fs] != 0, L);
  };
  const int b0 = lane * per, bc0 = min(b0, B - 1);
  int L0 = CELLS ? cells.L0 : ctx_len[bc0 * ms];
  int on0 = CELLS ? cells.on0 : 1;
  if (!CELLS && is_slow != nullptr) on0 = is_slow[bc0 * fs];
  __builtin_amdgcn_sched_barrier(0);
  // the guess: this workgroup's place if all sequences are equally long
  const int even = GUESS ? a.plan_even : 0;
  const int b_even = even > 0 ? j / even : B, slot_even = j - b_even * even;
  Tile T;
  if (GUESS && !PAGED && b_even < B) {
    Rows R;
    R.Kb = reinterpret_cast<const char*>(a.K + b_even * a.k_sb + h * a.k_sh);
    R.k_st = (uint32_t)a.k_st * 2u;
    R.k_lane = k_lane_of<false>(lane >> 4, lane & 15);
    R.n = lane & 15;
    issue_k_affine<false>(T, R, n_sink + (slot_even * kWaves + ((int)threadIdx.x >> 6)) * kTile, a.row_cap);
  }
  __builtin_amdgcn_sched_barrier(0);
  int L_0;
  const int t0 = tiles_of(b0, bc0, L0, on0, L_0);
  const int L_in_all = __builtin_amdgcn_readfirstlane(L0), L_all = __builtin_amdgcn_readfirstlane(L_0);
  bool same = even > 0 && (b0 >= B || (L0 == L_in_all && L_0 == L_all));
  int tiles = t0, count = t0 > 0;
  float least = t0 > 0 ? (float)t0 : 3e38f;
  for (int i = 1; i < per; ++i) {
    int L_in, L;
    const int t = lane_seq(i, L_in, L);
    same = same && (b0 + i >= B || (L_in == L_in_all && L == L_all));
    tiles += t;
    count += t > 0;
    least = t > 0 ? fminf(least, (float)t) : least;
  }
  if (GUESS && __all(same)) {
    if (b_even >= B) return;
    DenseShare sh;
    sh.bad = 0;
    view_of(b_even, L_in_all, sh.L, sh.recent, sh.bad);
    sh.first = slot_even * kWaves;
    sh.step = even * kWaves;
    sh.end = 1 << 30;
    sh.slot = slot_even;
    sh.n_rec = even;
    sh.have_k = !PAGED;
    if (slot_even == 0 && h == 0 && threadIdx.x == 0) a.seq_rec[b_even] = even;
    dense_body<EXPOSE, PAGED, true, false, true>(a, sh, h, b_even, T, lds, sc);
    return;
  }
  if (CELLS) {
    // above the sequences that take part (10 bits): this head's workgroups with a fast cell (10), those in front of this one
    // (10), and whether this is one (a launch has at most 256 cells; cells of a sequence lie 1 << row_lg workgroups apart)
    const int apart = 1 << cells.row_lg;
    for (int i = 0; i < per; ++i) {
      const int b = b0 + i, z = (b >> cells.row_lg) * (cells.n_split << cells.row_lg) + (b & (apart - 1));
      auto cells_below = [&](int w) { return min(max((w - z + apart - 1) >> cells.row_lg, 0), cells.n_split); };
      const int before = cells_below(j), here = cells_below(j + 1) - before;
      int L_in = L0, L;
      const int t = i == 0 ? t0 : lane_seq(i, L_in, L);
      count += b < B && t == 0 ? cells_below(W_max) << 10 | before << 20 | here << 30 : 0;
    }
  }
  const int inc_t = (int)wave_incl_scan((uint32_t)tiles), inc_c = (int)wave_incl_scan((uint32_t)count);
  PlanArgs p;
  p.total = __builtin_amdgcn_readlane(inc_t, 63);
  const uint32_t counts = __builtin_amdgcn_readlane(inc_c, 63);
  p.n_on = CELLS ? counts & 1023u : counts;
  if (a.slow_list != nullptr && h == 0 && j == 0 && threadIdx.x == 0) a.slow_list[0] = p.n_on;
  p.W = max(1, min(W_max, (int)((float)p.total * per_min)));
  if (p.total == 0) return;
  p.n_a = p.W;
  p.s_b = 1 << kShareLg;
  if (CELLS) {
    const int n_fast = (counts >> 10) & 1023u, fast_before = (counts >> 20) & 1023u, n_whole = W_max - n_fast;
    const bool fast = counts >> 30;
    // (a workgroup with a cell does cells.tiles * n_whole / W_max less than with equal shares)
    if (n_fast > 0 && cells.tiles * (float)n_whole > kLeastGain * (float)W_max) {
      // Smaller shares are at least plan_min tiles (and what the rounding of their size may take) and 1/16 of a whole one.
      const float t = (float)p.total, least_b = fmaxf(1.0625f * __builtin_amdgcn_rcpf(per_min) + 1.f, cells.tiles * (1.f / 15.f));
      const float over = t - (float)n_whole * cells.tiles;
      const int n_b = max(0, min(n_fast, (int)(over * __builtin_amdgcn_rcpf(least_b)) - n_whole));
      p.n_a = max(1, min(n_whole, (int)(t * per_min)));
      p.W = p.n_a + n_b;
      const float whole = (t + (float)n_b * cells.tiles) * __builtin_amdgcn_rcpf((float)p.W);
      if (n_b > 0) p.s_b = (int)((float)(1 << kShareLg) * (1.f - cells.tiles * __builtin_amdgcn_rcpf(whole)));
      j = fast ? p.n_a + fast_before : j - fast_before;
      if (!fast && j >= p.n_a) return;
    } else if (n_fast == 0) {  // head after head, as without cells (32 x 16384..65536 rows, G = 8: 1279 -> 1256 us a step)
      const int i = j * a.Hkv + h;
      h = i / W_max;
      j = i - h * W_max;
    }
  }
  if (j >= p.W) return;
  p.scale = (float)(share_start<CELLS>(p, p.W) - p.n_on) * __builtin_amdgcn_rcpf((float)p.total) * 0.999999f;
  p.h = -wave_max(-least) * p.scale > 2.f * kCross * p.scale + 8.f ? min((int)(0.5f * kCross * p.scale) + 1, 1 << (kShareLg - 2)) : 0;
  const int start = share_start<CELLS>(p, j);
  // the sequence at the share's start
  int before = inc_t - tiles, rank = inc_c - count;  // tiles, sequences in front of this lane's
  if (CELLS) rank &= 1023;
  int hit_i = -1, hit_P = 0, hit_rank = 0, hit_L = 0;
  for (int i = 0; i < per; ++i) {
    int L_in = L0;
    int off, L;
    const int t = i == 0 ? t0 : lane_seq(i, L_in, L);
    if (t > 0 && plan_border<CELLS>(p, before, rank, off) <= start && start < plan_border<CELLS>(p, before + t, rank + 1, off)) {
      hit_i = i;
      hit_P = before;
      hit_rank = rank;
      hit_L = L_in;
    }
    before += t;
    rank += t > 0;
  }
  const int src = __builtin_ctzll(__ballot(hit_i >= 0));
  int b = src * per + __builtin_amdgcn_readlane(hit_i, src), P = __builtin_amdgcn_readlane(hit_P, src);
  int r = __builtin_amdgcn_readlane(hit_rank, src), L_in = __builtin_amdgcn_readlane(hit_L, src);
  for (;;) {
    DenseShare sh;
    sh.bad = 0;
    const int t_b = view_of(b, L_in, sh.L, sh.recent, sh.bad);
    int g0, g1;
    const int x0 = plan_border<CELLS>(p, P, r, g0), x1 = plan_border<CELLS>(p, P + t_b, r + 1, g1);
    const int w0 = __builtin_amdgcn_readfirstlane(share_of<CELLS>(p, x0)), w1 = __builtin_amdgcn_readfirstlane(share_of<CELLS>(p, x1 - 1));
    sh.slot = j - w0;
    sh.n_rec = w1 - w0 + 1;
    // the tiles of the first workgroup and those in front of the last one, where they share with another sequence
    const int lo = x0 + g0, hi = x1 - g1;
    const float f = (float)t_b * __builtin_amdgcn_rcpf((float)(hi - lo));
    const bool part0 = w1 > w0 && x0 != share_start<CELLS>(p, w0), part1 = w1 > w0 && x1 != share_start<CELLS>(p, w1 + 1);
    auto tiles_to = [&](int w) { return min(t_b, (int)((float)(share_start<CELLS>(p, w) - lo) * f)); };  // in front of workgroup w's share
    const int A = part0 ? tiles_to(w0 + 1) : 0;
    const int Z = part1 ? tiles_to(w1) : t_b;
    // the workgroups that interleave with this one, and their tiles
    int full0 = w0 + part0, full1 = w1 + 1 - part1, a0 = A, z0 = Z;
    if (CELLS && full0 < p.n_a && p.n_a < full1) {
      if (j < p.n_a) full1 = p.n_a, z0 = tiles_to(p.n_a);
      else full0 = p.n_a, a0 = tiles_to(p.n_a);
    }
    int first, step = kWaves, end;
    if (part0 && sh.slot == 0) {
      first = 0;
      end = A;
    } else if (part1 && j == w1) {
      first = Z;
      end = t_b;
    } else {
      first = a0 + (j - full0) * kWaves;
      step = (full1 - full0) * kWaves;
      end = z0;
    }
    sh.first = __builtin_amdgcn_readfirstlane(first);
    sh.step = __builtin_amdgcn_readfirstlane(step);
    sh.end = __builtin_amdgcn_readfirstlane(end);
    if (sh.slot == 0 && h == 0 && threadIdx.x == 0) {
      a.seq_rec[b] = sh.n_rec;
      if (a.slow_list != nullptr)
        reinterpret_cast<int4*>(a.slow_list)[1 + r] = make_int4(b, min(max(L_in, 0), len_cap), sh.n_rec, 0);
    }
    // A zero the compiler cannot see through: without it everything the body derives from the thread index is
    // computed once in front of this loop and kept in registers across the body.
    int zero = 0;
    asm volatile("" : "+s"(zero));
    sh.have_k = false;
    dense_body<EXPOSE, PAGED, true, false, true>(a, sh, h, b, T, lds, sc, zero);
    P += t_b;
    if (__builtin_amdgcn_readfirstlane(x1) >= share_start<CELLS>(p, j + 1)) return;
    do {  // (there is one: the list goes on)
      ++b;
    } while (is_slow != nullptr && is_slow[b * fs] == 0);
    ++r;
    L_in = ctx_len[b * ms];
    __syncthreads();  // the combine of this sequence is read before the next one's logits go into the same LDS
  }
}
template <int EXPOSE, bool PAGED>
__global__ __launch_bounds__(kAttnThreads, 1) void attn_dense_planned_kernel(const int32_t* ctx_len, const uint8_t* is_slow, const int32_t* q_len,
                                                                             uint32_t strides, int B, int W_max, float per_min, int n_sink,
                                                                             int recent_in, int len_cap, const AttnArgs a) {
  __shared__ __align__(16) float s_patch[kWaves * patch_floats(EXPOSE, true)];
  Scored sc = scored_of(s_patch);
  planned_body<EXPOSE, PAGED, true>(blockIdx.y, blockIdx.x, ctx_len, is_slow, q_len, strides, B, W_max, per_min, n_sink, recent_in, len_cap, a,
                                    s_patch, sc);
  if (EXPOSE >= 3) score_tail<EXPOSE == 4>(a, sc, s_patch);
}

// ------------------------------------------------------------------------------------------------
// evidence kernel: the logits of one query over the allowed set J (and the key norms), and their softmax statistics;
// no V row is read.  This is a query of a window: the next launches read the same K rows, so their loads leave them to the
// caches instead of streaming past them (16 queries over 58 MB of K: 309 us streamed, 274 not), as long as the caches can hold them.
// LINES, for a K that may be larger: left to the caches such a K pushes out the logits and the accumulator, which the
// accumulation behind this launch then fetches from memory (32 x 16000 rows, 8 KV heads, one head each: 13.9 us, streamed 12.1), and
// streamed in pieces of half a line, as the product wants them, a line may be gone before its other half is asked for
// (210 us; from the caches 193).  So a request is 8 whole lines of 8 rows, streamed (175), and lanes n and n ^ 8 swap what they got
// for each other: 32 register moves a tile, from there on the layout is the other's.  Whether K fits, the kernel finds by
// adding up the lengths, which only the device knows: up to a.cached_rows the same requests go through the caches, as a wave's
// first two tiles do in any case.
// Windows of 8 queries, 16000 rows, 8 KV heads, us, plain requests / this: G = 4, 10 sequences (312 MB) 568 / 509, 12 (375) 681 / 581, 16 (500) 914 / 756;
// G = 1, 493 / 453, 619 / 515, 835 / 668; 16 x 4000..16000 (312) 628 / 534.  All streamed although K fits: 6 sequences (188) 305 / 337, 8 (250) 414 / 457,
// 9 (281) 459 / 489.  A launch whose bound fits stays with the plain requests: 4 sequences 221, G = 1 203, with norms 237; by lines 224, 207, 244.
// What bounds it: the rows, at the rate the last-level cache gives them (58 MB: loads alone 10.0 us behind a launch of
// 1.6 us).  So every wave has two tiles on their way all the time, each refilled when its products are done; the
// statistics are kept per lane (its own positions of its head) and meet once at the end, so that nothing in the loop
// crosses lanes; the code is a loop of one step, and the first tile is requested from arguments in registers.  The two
// tiles lie a workgroup's stride apart: as neighbours (16 KB in one piece per wave) they take 13 % longer.
// Against the dense kernel without its V half, which this replaces, us per query with the accumulation behind it, 8 KV heads: 2 sequences of
// 12000..16384 rows with norms 19.9 -> 17.0; 2 x 4096 11.7 -> 9.6; 8 x 8000..16000 51.7 -> 42.6; 1 x 130000 54.6 -> 45.1.
// With the head as the first index of both launches, so that the accumulation finds the logits in its L2, on another box: 15.86 -> 15.52, 7.85 -> 7.45,
// 41.3 -> 39.4, 48.8 -> 48.4; 32 x 512..4000, two heads a group 34.2 -> 31.2.
// ------------------------------------------------------------------------------------------------
constexpr int kEvidenceStash = 2432;  // floats of logits a wave parks in LDS: four tiles of 16 heads and norms, 15 of 4 heads and norms
struct KPair {    // two tiles of K: tile hf is blocks 2 hf and 2 hf + 1
  uint4 k[4][4];  // block i: row 16 (i & 1) + n of its tile, dims kb * 32 + 8 * jg .. + 8
                  // (LINES, until swapped: row 16 (i & 1) + 8 (kb & 1) + (n & 7), dims (kb / 2) * 64 + 32 * (n / 8) + 8 * jg .. + 8)
};
// Within a row of 16 lanes: the value of lane n & 7, or of lane 8 + (n & 7).
__device__ __forceinline__ int lower_half(int v) { return __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0xc, false); }
__device__ __forceinline__ int upper_half(int v) { return __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0x3, false); }
// Two requests for whole lines become two operands: lanes n >= 8 trade their x for the y of lane n - 8.
__device__ __forceinline__ void swap_halves(uint32_t& x, uint32_t& y) {
  const int a = (int)x, b = (int)y;
  x = (uint32_t)__builtin_amdgcn_update_dpp(a, b, 0x128, 0xf, 0xc, false);
  y = (uint32_t)__builtin_amdgcn_update_dpp(b, a, 0x128, 0xf, 0x3, false);
}
__device__ __forceinline__ void swap_halves(uint4& x, uint4& y) {
  swap_halves(x.x, y.x);
  swap_halves(x.y, y.y);
  swap_halves(x.z, y.z);
  swap_halves(x.w, y.w);
}
template <int EXPOSE, bool PAGED, bool LINES>
__global__ __launch_bounds__(kAttnThreads, 3) void attn_evidence_kernel(const uint16_t* K, const int32_t* ctx_len, const int32_t* q_len,
                                                                        const int64_t k_sb, const int64_t k_sh, const uint32_t k_st,
                                                                        const int n_sink, const int row_cap, const int len_cap,
                                                                        const AttnArgs a) {
  typedef typename RowOff<PAGED>::type OffT;
  __shared__ __align__(16) float s_stash[kWaves][kEvidenceStash];
  __shared__ __align__(16) float s_m[16][kWaves], s_l[16][kWaves];
  const int h = blockIdx.x, slot = blockIdx.y, b = blockIdx.z;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jg = lane >> 4, n = lane & 15;
  const char* const Kb = reinterpret_cast<const char*>(K + b * k_sb + h * k_sh);
  const uint32_t k_lane = LINES ? (n >> 3) * 64 + jg * 16 : jg * 16;
  const int first = slot * kWaves + w;
  int bad = 0;
  Pages P;
  int pg[4], pg_row[4];  // PAGED: block-table entries of the unit's rows and the rows they were read for
  auto pages_for = [&](int hf, int t, int hi) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      pg_row[2 * hf + i] = (int)min((uint32_t)n_sink + (uint32_t)(t * kTile + 16 * i + n), (uint32_t)hi);
      pg[2 * hf + i] = P.page_of(pg_row[2 * hf + i]);
    }
  };
  // rows of tile t into half hf; rows above hi (no position of J) read row hi, whose block is a valid one
  bool stream = false;  // LINES, the same for all workgroups once the lengths are known
  auto issue = [&](KPair& U, int hf, int t, int hi) {
    auto row_at = [&](int i) { return (int)min((uint32_t)n_sink + (uint32_t)(t * kTile + i), (uint32_t)hi); };  // (n_sink is not bounded)
    auto offset = [&](int row) { return (OffT)((OffT)(uint32_t)row * k_st + k_lane); };
    if constexpr (LINES) {
      OffT o[4];  // rows 8 j + (n & 7)
      if (PAGED) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int row = P.phys(pg_row[2 * hf + i], pg[2 * hf + i], bad);
          o[2 * i] = offset(lower_half(row));
          o[2 * i + 1] = offset(upper_half(row));
        }
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = offset(row_at(8 * j + (n & 7)));
      }
      auto request = [&](auto past_caches) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int l = 0; l < 2; ++l) U.k[2 * hf + (j >> 1)][2 * l + (j & 1)] = load_row16<decltype(past_caches)::value>(Kb, o[j], l * 128);
      };
      if (stream) request(std::integral_constant<bool, true>());  // (wave-uniform, as many loads on either side)
      else request(std::integral_constant<bool, false>());
    } else {
      OffT o[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) o[i] = offset(PAGED ? P.phys(pg_row[2 * hf + i], pg[2 * hf + i], bad) : row_at(16 * i + n));
#pragma unroll
      for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int i = 0; i < 2; ++i) U.k[2 * hf + i][kb] = load_row16<false>(Kb, o[i], kb * 64);
    }
  };
  KPair U;
  // The first tile's rows follow from the arguments that the wave finds in registers (a paged cache's from the length on).
  if (!PAGED) issue(U, 0, first, row_cap);
  const int L_in = ctx_len[b];
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(a.q), "s"(a.logits), "s"(a.part), "s"(a.guard), "s"(a.ld_pos), "s"(a.Hq), "s"(a.Hkv), "s"(a.G), "s"(a.recent), "s"(a.n_split),
               "s"(a.scale_log2));
  const int G = a.G;
  const int64_t head0 = (int64_t)b * a.Hq + h * G;
  const int step = a.n_split * kWaves;
  if (!PAGED) issue(U, 1, first + step, row_cap);
  bf16x8 qreg[4];
  load_q_raw(qreg, a.q, head0, G, jg, n);
  int L, recent;
  window_view(q_len, b, guarded_len(L_in, len_cap, bad), a.recent, L, recent);
  const int NJ = max(0, L - recent - n_sink);
  const int nT = (NJ + kTile - 1) / kTile;
  const int hi = max(n_sink + NJ - 1, 0);
  if (PAGED && first < nT) {
    P = pages_of(a, b, L);
    pages_for(0, first, hi);
    pages_for(1, first + step, hi);
    issue(U, 0, first, hi);
    issue(U, 1, first + step, hi);
    pages_for(0, first + 2 * step, hi);
    pages_for(1, first + 3 * step, hi);
  }
  mask_q(qreg, G, n);

  const int rows_exp = G + (EXPOSE == 2 ? 1 : 0);
  const int tile_f = rows_exp * kTile;
  const int stash_cap = kEvidenceStash / tile_f;
  float* const stash = &s_stash[w][0];
  float* const lg = a.logits + (int64_t)(b * a.Hkv + h) * rows_exp * a.ld_pos;
  int n_stashed = 0, k_flushed = 0;
  auto flush = [&]() {
    __builtin_amdgcn_wave_barrier();
    const int n_f4 = n_stashed * (tile_f / 4);
    for (int f = lane; f < n_f4; f += 64) {
      const int i = f / (tile_f / 4), rem = f - i * (tile_f / 4);
      const int t = first + (k_flushed + i) * step;
      *reinterpret_cast<float4*>(lg + ((int64_t)t * tile_f + rem * 4)) = *reinterpret_cast<const float4*>(stash + f * 4);
    }
    __builtin_amdgcn_wave_barrier();
    k_flushed += n_stashed;
    n_stashed = 0;
  };
  // statistics of the positions this lane has seen (the four lanes of a head meet at the end)
  float m_run = kNeg, l_run = 0.f;
  // tiles t and t + step; the second may lie past the end, then it counts for nothing
  auto pair_step = [&](int t, auto refill) {
    float y[4][4];
    float k2[4];  // (lanes with jg == n / 4) squared norm of row 16 i + n: the diagonal of K K^T
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (LINES) {
        swap_halves(U.k[i][0], U.k[i][1]);
        swap_halves(U.k[i][2], U.k[i][3]);
      }
      f32x4 s = {0.f, 0.f, 0.f, 0.f}, d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(U.k[i][kb]), qreg[kb], s, 0, 0, 0);
        if (EXPOSE == 2) d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(U.k[i][kb]), as_bf16x8(U.k[i][kb]), d, 0, 0, 0);
      }
      if (EXPOSE == 2) k2[i] = (n & 3) == 0 ? d[0] : (n & 3) == 1 ? d[1] : (n & 3) == 2 ? d[2] : d[3];
#pragma unroll
      for (int j = 0; j < 4; ++j) y[i][j] = s[j] * a.scale_log2;
      if (decltype(refill)::value && (i & 1) != 0) {
        issue(U, i >> 1, t + (2 + (i >> 1)) * step, hi);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (decltype(refill)::value && PAGED) {
      pages_for(0, t + 4 * step, hi);
      pages_for(1, t + 5 * step, hi);
    }
    float m_new = m_run;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      if (hf == 1 && t + step >= nT) break;
      float* st = stash + n_stashed * tile_f;
#pragma unroll
      for (int i = 2 * hf; i < 2 * hf + 2; ++i) {
        // (positions past |J| land in the padding, never used)
        float* row = st + (i & 1) * 16;
        if (n < G) *reinterpret_cast<float4*>(row + n * kTile + 4 * jg) = make_float4(y[i][0], y[i][1], y[i][2], y[i][3]);
        if (EXPOSE == 2 && jg == (n >> 2)) row[G * kTile + n] = k2[i];
      }
      if (++n_stashed == stash_cap) flush();
    }
    bool ok[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ok[i][j] = (t + (i >> 1) * step) * kTile + 16 * (i & 1) + 4 * jg + j < NJ;
        m_new = fmaxf(m_new, ok[i][j] ? y[i][j] : kNeg);
      }
    l_run *= fast_exp2(m_run - m_new);
    m_run = m_new;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) l_run += ok[i][j] ? fast_exp2(y[i][j] - m_new) : 0.f;
  };
  if (first < nT) {
    if (LINES) {
      float rows = 0.f;
      for (int i = lane; i < a.plan_batch; i += 64) rows += (float)min(max(ctx_len[i], 0), len_cap);
      stream = __builtin_amdgcn_readfirstlane(wave_sum_f(rows) > (float)a.cached_rows) != 0;
    }
    int t = first;
    for (; t + 2 * step < nT; t += 2 * step) pair_step(t, std::integral_constant<bool, true>());
    pair_step(t, std::integral_constant<bool, false>());
    flush();
  }
  const float M = rows_max(m_run);
  const float l = rows_sum(l_run * fast_exp2(m_run - M));
  if (lane < 16) {
    s_m[lane][w] = M;
    s_l[lane][w] = l;
  }
  __syncthreads();
  if ((int)threadIdx.x < G) {  // the record's header: no output, and nothing beyond J
    const float4 m4 = *reinterpret_cast<const float4*>(&s_m[threadIdx.x][0]), l4 = *reinterpret_cast<const float4*>(&s_l[threadIdx.x][0]);
    const float Mw = fmaxf(fmaxf(m4.x, m4.y), fmaxf(m4.z, m4.w));
    const float lw = l4.x * fast_exp2(m4.x - Mw) + l4.y * fast_exp2(m4.y - Mw) + l4.z * fast_exp2(m4.z - Mw) + l4.w * fast_exp2(m4.w - Mw);
    *reinterpret_cast<float4*>(a.part + ((head0 + threadIdx.x) * kSlotCap + slot) * kPartStride) = make_float4(Mw, lw, Mw, lw);
  }
  report_guard(a.guard, bad);
}
hipError_t launch_attn_evidence(const AttnArgs& a, int B, int n_slots, hipStream_t s) {
  const dim3 grid(a.Hkv, n_slots, B), block(kAttnThreads);  // heads first: Place in sfi_select.hip
#define SFI_EVIDENCE_L(EXPOSE, PAGED, LINES)                                                                                     \
  hipLaunchKernelGGL((attn_evidence_kernel<EXPOSE, PAGED, LINES>), grid, block, 0, s, a.K, a.ctx_len, a.q_len, a.k_sb, a.k_sh,    \
                     (uint32_t)a.k_st * 2u, a.n_sink, a.row_cap, a.len_cap, a)
#define SFI_EVIDENCE(EXPOSE, PAGED)                          \
  do {                                                       \
    if (a.cached_rows > 0) SFI_EVIDENCE_L(EXPOSE, PAGED, true); \
    else SFI_EVIDENCE_L(EXPOSE, PAGED, false);               \
  } while (0)
  if (a.table != nullptr) {
    if (a.with_knorm) SFI_EVIDENCE(2, true);
    else SFI_EVIDENCE(1, true);
  } else {
    if (a.with_knorm) SFI_EVIDENCE(2, false);
    else SFI_EVIDENCE(1, false);
  }
#undef SFI_EVIDENCE
#undef SFI_EVIDENCE_L
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// gather kernel: each wave walks tiles first, first + step, ... of its list with the dense kernel's loop: one tile
// buffer whose K half is refilled with the next tile's rows right after S^T, the V half right after P V; the selected
// indices are read two tiles ahead.  Loads past the wave's last tile fall on row 0 (no branch around a load, so every
// wait names exactly the loads it needs).  A launch whose split leaves every wave at most one tile skips the loop.
//
// A short launch is its chain of round trips: kernel arguments, then the step's scalars and the first indices, then the
// rows.  The first argument load of a wave takes 0.5 us, so what the second link needs travels in the leading scalar
// arguments, which the hardware hands to the wave in registers (-amdgpu-kernarg-preload-count); the rest of the
// arguments arrives while the indices are on their way.  Nothing waits for q before the rows are requested, and no
// division stands in the way (a vector instruction of a lone wave takes 1.7 us per thousand).  Measured with this order
// against arguments read where they are used and q masked where it is loaded: 131072 rows / 8 KV heads 9.6 -> 9.0 us,
// 4 x 32768 rows 11.1 -> 10.6 us, 4096 rows / 2 KV heads 6.4 -> 5.6 us.
// ------------------------------------------------------------------------------------------------
// The preloaded arguments: shape, see fast_cell.
template <bool PAGED, bool WIDE, bool LOCAL>
__device__ __forceinline__ void gather_body(const FastCell& cell, const int32_t* sel_idx, const int32_t* n_sel_p, const int32_t* ctx_len_p,
                                            const int32_t* recent_start_p, const uint8_t* is_slow_p, const uint32_t sel_stride,
                                            const uint32_t shape, const int n_sink, const int n_split, const AttnArgs& a, float* lds) {
  const int slot = cell.slot, h = cell.h, b = cell.b;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jg = lane >> 4, n = lane & 15;
  const int bh = b * (int)(shape & 0xffffu) + h;
  const int bm = b << ((shape >> 16) & 15u);
  const bool flagged = ((shape >> 20) & 1u) != 0u;
  const int first = slot * kWaves + w, step = n_split * kWaves;
  const int p_first = first * kTile, pstep = step * kTile;
  // First round of loads, none depending on another: the scalars and the flag, the indices of the first tile (read before
  // the list length is known, clamped to the row of sel_idx), and the arguments that come from memory.
  const int L_in = ctx_len_p[bm], n_sel_in = n_sel_p[bh], rs_in = recent_start_p[bm];
  ListWalk W;
  W.sel = sel_idx + (int64_t)bh * sel_stride;
  W.sel_cap = max((int)sel_stride - 1, 0);  // sel_stride = 0: the host points sel_idx at one readable word
  W.n_sink = n_sink;
  const int slow = is_slow_p[flagged ? (uint32_t)b << (2u * ((shape >> 16) & 15u)) : 0u];  // (a readable byte in any case)
  const int sA = W.sel_at_nonempty(p_first + n), sB = W.sel_at_nonempty(p_first + 16 + n);
  __builtin_amdgcn_sched_barrier(0);
  // everything uniform is asked for before the first of it is used: one wait
  asm volatile("" ::"s"(L_in), "s"(n_sel_in), "s"(rs_in), "s"(a.q), "s"(a.K), "s"(a.V), "s"(a.k_sb), "s"(a.k_sh), "s"(a.k_st),
               "s"(a.v_sb), "s"(a.v_sh), "s"(a.v_st), "s"(a.Hq), "s"(a.G), "s"(a.scale_log2), "s"(a.len_cap));
  if (PAGED) asm volatile("" ::"s"(a.table), "s"(a.table_stride), "s"(a.page_lg), "s"(a.page_rpb), "s"(a.n_blocks));
  const int G = a.G;
  const int64_t head0 = (int64_t)b * a.Hq + h * G;
  bf16x8 qreg[4];
  load_q_raw<WIDE>(qreg, a.q, head0, G, jg, n);
  Rows R;
  R.Kb = reinterpret_cast<const char*>(a.K + b * a.k_sb + h * a.k_sh);
  R.Vb = reinterpret_cast<const char*>(a.V + b * a.v_sb + h * a.v_sh);
  R.k_st = (uint32_t)a.k_st * 2u;
  R.v_st = (uint32_t)a.v_st * 2u;
  R.k_lane = k_lane_of<WIDE>(jg, n);
  R.v_lane = n * 16;
  R.jg = jg;
  R.n = n;
  W.bad = 0;
  const int L = guarded_len(L_in, a.len_cap, W.bad);
  W.set_counts(L, n_sel_in, rs_in, (int)sel_stride);
  const int nT = (W.N + kTile - 1) / kTile;
  asm volatile("" ::"s"(R.Kb), "s"(R.Vb), "s"(W.nS), "s"(W.nSel), "s"(W.rs), "s"(W.N), "s"(nT));  // worked out while the indices travel
  __builtin_amdgcn_sched_barrier(0);
  if (flagged && __builtin_amdgcn_readfirstlane(slow) != 0) return;

  Tile T;
  float m_run = kNeg, l_run = 0.f;
  f32x4 acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Memory instructions go out in the same order here as in an iteration of the loop below -- K rows,
  // the indices of the tile after, V rows -- so the in-order load counter reads the same on both ways
  // into the loop.  A wave without tiles reads row 0 and skips the loop.
  // PAGED adds one stage to the pipeline: indices are read two tiles ahead, the block-table entries
  // of the rows they name one tile ahead (order: K rows, table entries, indices, V rows).
  int sAn, sBn;            // !PAGED: indices of the next tile; PAGED: of the tile after the next
  int ra_n = 0, rb_n = 0;  // PAGED: logical rows of the next tile and their block-table entries
  int pa_n = 0, pb_n = 0;
  Pages P;
  if (PAGED) {
    P = pages_of(a, b, L);
    const int sA1 = W.sel_at_nonempty(p_first + pstep + n), sB1 = W.sel_at_nonempty(p_first + pstep + 16 + n);
    int ra = W.row_of(p_first + n, sA), rb = W.row_of(p_first + 16 + n, sB);
    ra = P.phys(ra, P.page_of(ra), W.bad);
    rb = P.phys(rb, P.page_of(rb), W.bad);
    __builtin_amdgcn_sched_barrier(0);
    issue_k_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
    __builtin_amdgcn_sched_barrier(0);
    ra_n = W.row_of(p_first + pstep + n, sA1);
    rb_n = W.row_of(p_first + pstep + 16 + n, sB1);
    pa_n = P.page_of(ra_n);
    pb_n = P.page_of(rb_n);
    __builtin_amdgcn_sched_barrier(0);
    sAn = W.sel_at_nonempty(p_first + 2 * pstep + n);
    sBn = W.sel_at_nonempty(p_first + 2 * pstep + 16 + n);
    __builtin_amdgcn_sched_barrier(0);
    issue_v_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
    __builtin_amdgcn_sched_barrier(0);
  } else {
    const int ra = W.row_of(p_first + n, sA), rb = W.row_of(p_first + 16 + n, sB);
    __builtin_amdgcn_sched_barrier(0);  // the compiler's scheduler must not reorder the three groups
    issue_k_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
    __builtin_amdgcn_sched_barrier(0);
    sAn = W.sel_at_nonempty(p_first + pstep + n);
    sBn = W.sel_at_nonempty(p_first + pstep + 16 + n);
    __builtin_amdgcn_sched_barrier(0);
    issue_v_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
    __builtin_amdgcn_sched_barrier(0);
  }
  mask_q<WIDE>(qreg, G, n);
  // The last tile is taken after the loop, without the refill: no rows are requested for a tile that does not
  // exist, and nothing is in flight when the wave reaches the record write (worth 0.05 us at most: the tail
  // waits for its own stores far longer than for such rows).
  int p0 = p_first;
  for (int t = first; t + step < nT; t += step) {
    const int pn = p0 + pstep;
    float y[8];
    qk_phase<WIDE>(T, qreg, a.scale_log2, y);
    int ra, rb;
    if (PAGED) {
      ra = P.phys(ra_n, pa_n, W.bad);
      rb = P.phys(rb_n, pb_n, W.bad);
      issue_k_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
      ra_n = W.row_of(pn + pstep + n, sAn);  // row 0 past the list
      rb_n = W.row_of(pn + pstep + 16 + n, sBn);
      pa_n = P.page_of(ra_n);
      pb_n = P.page_of(rb_n);
      sAn = W.sel_at_nonempty(pn + 2 * pstep + n);
      sBn = W.sel_at_nonempty(pn + 2 * pstep + 16 + n);
    } else {
      ra = W.row_of(pn + n, sAn);  // row 0 past the list
      rb = W.row_of(pn + 16 + n, sBn);
      issue_k_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
      sAn = W.sel_at_nonempty(pn + pstep + n);
      sBn = W.sel_at_nonempty(pn + pstep + 16 + n);
    }
    if (p0 + kTile > W.N) mask_tail<WIDE>(T, y, jg, p0, W.N);
    bf16x8 a_hi, a_lo;
    softmax_phase(y, acc, m_run, l_run, jg, a_hi, a_lo);
    pv_phase(T, a_hi, a_lo, acc);
    issue_v_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
    p0 = pn;
  }
  if (first < nT) {
    float y[8];
    qk_phase<WIDE>(T, qreg, a.scale_log2, y);
    if (p0 + kTile > W.N) mask_tail<WIDE>(T, y, jg, p0, W.N);
    bf16x8 a_hi, a_lo;
    softmax_phase(y, acc, m_run, l_run, jg, a_hi, a_lo);
    pv_phase(T, a_hi, a_lo, acc);
  }
  const WgOut o = wg_out_of(a, bh);
  if (finish_wg<false, WIDE ? 1 : 2, LOCAL>(o, head0, G, slot, acc, m_run, rows_sum(l_run), lds, (WIDE ? 8 : 16) * kHeadDim)) {
    m_run = kNeg;
    l_run = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int p = 0; p < W.N; p += kTile) {
      int ra = W.row_of(p + n, W.sel_at_nonempty(p + n)), rb = W.row_of(p + 16 + n, W.sel_at_nonempty(p + 16 + n));
      if (PAGED) {
        ra = P.phys(ra, P.page_of(ra), W.bad);
        rb = P.phys(rb, P.page_of(rb), W.bad);
      }
      issue_rows<typename RowOff<PAGED>::type, WIDE>(T, R, ra, rb);
      float y[8];
      qk_phase<WIDE>(T, qreg, a.scale_log2, y);
      if (p + kTile > W.N) mask_tail<WIDE>(T, y, jg, p, W.N);
      bf16x8 a_hi, a_lo;
      softmax_phase(y, acc, m_run, l_run, jg, a_hi, a_lo);
      pv_phase(T, a_hi, a_lo, acc);
    }
    store_heads(o, head0, G, acc, l_run);
  }
  report_guard(a.guard, W.bad);  // last: the way to the record and the merge is the launch's critical path
}
template <bool PAGED, bool WIDE, bool LOCAL>
__global__ __launch_bounds__(kAttnThreads, 3) void attn_gather_kernel(const int32_t* sel_idx, const int32_t* n_sel_p, const int32_t* ctx_len_p,
                                                                      const int32_t* recent_start_p, const uint8_t* is_slow_p,
                                                                      const uint32_t sel_stride, const uint32_t shape, const int n_sink,
                                                                      const int n_split, const AttnArgs a) {
  const FastCell cell = fast_cell<LOCAL>(shape);
  if (cell.off) return;
  __shared__ __align__(16) float s_red[kWaves * (WIDE ? 8 : 16) * kHeadDim];
  gather_body<PAGED, WIDE, LOCAL>(cell, sel_idx, n_sel_p, ctx_len_p, recent_start_p, is_slow_p, sel_stride, shape, n_sink, n_split, a, s_red);
}

// ------------------------------------------------------------------------------------------------
// Memory skeleton of the fast step -- a measurement aid, not part of the path.  Same grid, same three
// scalars, same index loads and the same row loads as the gather kernels, but no arithmetic: what
// arrives is folded into one word per lane.  It answers what a launch of this shape costs when the
// matrix and vector units do nothing, i.e. the floor the real kernel can be held against.
//   TAIL   the workgroup's record goes through the same LDS combine, device-scope record stores,
//          arrival counter and last-workgroup merge as in the real kernel (the numbers are junk);
//          without it every workgroup ends with one plain 4-byte store.
//   BURST  instead of walking its tiles with one register buffer (K half and V half refilled as the
//          real loop does), a wave requests the rows of all its tiles at once, straight into LDS
//          (global_load_lds, 16 bytes per lane), and waits once: the most requests in flight the
//          launch shape allows.  The workgroup owns tiles [slot * tpw, (slot + 1) * tpw) of the list,
//          wave w the tiles w, w + 4, ... of that range; tpw * 16 KB of dynamic LDS.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ uint32_t fold16(const uint4& v) { return v.x ^ v.y ^ v.z ^ v.w; }

//   depth  1: stop after the scalars and indices; 2: load nothing at all (the cost of the bare launch).
// The leading arguments are the gather kernel's: they arrive in registers, and the scalars and the first indices are
// requested from them before the arguments that come from memory are asked for.
template <bool WIDE, int TAIL, bool BURST>  // TAIL 2: as LOCAL
__global__ __launch_bounds__(kAttnThreads, BURST ? 1 : 3) void attn_gather_floor_kernel(const int32_t* sel_idx, const int32_t* n_sel_p,
                                                                                        const int32_t* ctx_len_p, const int32_t* recent_start_p,
                                                                                        const uint8_t*, const uint32_t sel_stride,
                                                                                        const uint32_t shape, const int n_sink,
                                                                                        const int n_split, const AttnArgs a, int tpw,
                                                                                        int depth) {
  extern __shared__ uint4 s_rows[];  // BURST: [tpw][16 instructions][64 lanes]
  const FastCell cell = fast_cell<TAIL == 2>(shape);
  if (cell.off) return;
  const int slot = cell.slot, h = cell.h, b = cell.b;
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jg = lane >> 4, n = lane & 15;
  const int bh = b * (int)(shape & 0xffffu) + h;
  const int bm = b << ((shape >> 16) & 15u);
  uint32_t fold = 0u;
  if (TAIL == 0 && !BURST && depth == 2) {  // wave-uniform: the bare launch
    const int64_t head0 = (int64_t)b * a.Hq + h * a.G;
    if (lane == 0) reinterpret_cast<uint32_t*>(a.part)[((head0 * a.slot_cap + slot) * kPartStride) + w] = (uint32_t)slot;
    return;
  }
  const int p_first = (BURST ? slot * tpw + w : slot * kWaves + w) * kTile;
  const int L_in = ctx_len_p[bm], n_sel_in = n_sel_p[bh], rs_in = recent_start_p[bm];
  ListWalk W;
  W.sel = sel_idx + (int64_t)bh * sel_stride;
  W.sel_cap = max((int)sel_stride - 1, 0);
  W.n_sink = n_sink;
  W.bad = 0;
  const int sA0 = W.sel_at_nonempty(p_first + n), sB0 = W.sel_at_nonempty(p_first + 16 + n);
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(L_in), "s"(n_sel_in), "s"(rs_in), "s"(a.K), "s"(a.V), "s"(a.k_sb), "s"(a.k_sh), "s"(a.k_st), "s"(a.v_sb),
               "s"(a.v_sh), "s"(a.v_st), "s"(a.Hq), "s"(a.G), "s"(a.len_cap));
  const int G = a.G;
  const int64_t head0 = (int64_t)b * a.Hq + h * G;
  Rows R;
  R.Kb = reinterpret_cast<const char*>(a.K + b * a.k_sb + h * a.k_sh);
  R.Vb = reinterpret_cast<const char*>(a.V + b * a.v_sb + h * a.v_sh);
  R.k_st = (uint32_t)a.k_st * 2u;
  R.v_st = (uint32_t)a.v_st * 2u;
  R.k_lane = k_lane_of<WIDE>(jg, n);
  R.v_lane = n * 16;
  R.jg = jg;
  R.n = n;
  if (TAIL == 0 && !BURST && depth == 1) {  // wave-uniform: scalars and the first tile's indices, nothing else
    fold = (uint32_t)(L_in ^ n_sel_in ^ rs_in ^ sA0 ^ sB0);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) fold ^= __shfl_xor(fold, d);
    if (lane == 0) reinterpret_cast<uint32_t*>(a.part)[((head0 * a.slot_cap + slot) * kPartStride) + w] = fold;
    return;
  }
  if (BURST) {
    // indices of all of this wave's tiles (rows n and 16 + n of each)
    constexpr int kMaxT = 4;  // tiles per wave: tpw <= 16
    int sA[kMaxT], sB[kMaxT];
    sA[0] = sA0;
    sB[0] = sB0;
#pragma unroll
    for (int k = 1; k < kMaxT; ++k) {
      const int p0 = p_first + kWaves * k * kTile;
      sA[k] = W.sel_at_nonempty(p0 + n);
      sB[k] = W.sel_at_nonempty(p0 + 16 + n);
    }
    const int L = guarded_len(L_in, a.len_cap, W.bad);
    W.set_counts(L, n_sel_in, rs_in, (int)sel_stride);
    const int nT = (W.N + kTile - 1) / kTile;
#pragma unroll
    for (int k = 0; k < kMaxT; ++k) {
      const int lt = w + kWaves * k;            // tile within the workgroup's range
      const int t = slot * tpw + lt;
      if (lt < tpw && t < nT) {                 // wave-uniform
        const int p0 = t * kTile;
        const int ra = W.row_of(p0 + n, sA[k]), rb = W.row_of(p0 + 16 + n, sB[k]);
        uint4* dst = s_rows + (size_t)lt * 16 * 64;
#pragma unroll
        for (int i = 0; i < 8; ++i) {           // instruction i: rows 4 i .. 4 i + 3 of the tile, 16 lanes x 16 bytes each
          const int row = __shfl(i < 4 ? ra : rb, (4 * i + jg) & 15);  // resolved by the lane that holds that position
          const char* gk = R.Kb + (size_t)((uint32_t)row * R.k_st + (uint32_t)n * 16u);
          const char* gv = R.Vb + (size_t)((uint32_t)row * R.v_st + (uint32_t)n * 16u);
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gk,
                                           (__attribute__((address_space(3))) void*)(dst + i * 64), 16, 0, 0);
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)gv,
                                           (__attribute__((address_space(3))) void*)(dst + (8 + i) * 64), 16, 0, 0);
        }
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): every row of this wave has landed in LDS
#pragma unroll
    for (int k = 0; k < kMaxT; ++k) {
      const int lt = w + kWaves * k;
      const int t = slot * tpw + lt;
      if (lt < tpw && t < nT) {
        const uint4* src = s_rows + (size_t)lt * 16 * 64;
        for (int i = 0; i < 16; ++i) fold ^= fold16(src[i * 64 + lane]);
      }
    }
  } else {
    const int first = slot * kWaves + w, step = n_split * kWaves;
    const int pstep = step * kTile;
    const int L = guarded_len(L_in, a.len_cap, W.bad);
    W.set_counts(L, n_sel_in, rs_in, (int)sel_stride);
    Tile T;
    const int nT = (W.N + kTile - 1) / kTile;
    asm volatile("" ::"s"(R.Kb), "s"(R.Vb), "s"(W.nS), "s"(W.nSel), "s"(W.rs), "s"(W.N), "s"(nT));  // as the kernel does
    __builtin_amdgcn_sched_barrier(0);
    int ra = W.row_of(p_first + n, sA0), rb = W.row_of(p_first + 16 + n, sB0);
    __builtin_amdgcn_sched_barrier(0);
    issue_k_rows<uint32_t, WIDE>(T, R, ra, rb);
    __builtin_amdgcn_sched_barrier(0);
    int sAn = W.sel_at_nonempty(p_first + pstep + n), sBn = W.sel_at_nonempty(p_first + pstep + 16 + n);
    __builtin_amdgcn_sched_barrier(0);
    issue_v_rows<uint32_t, WIDE>(T, R, ra, rb);
    __builtin_amdgcn_sched_barrier(0);
    int pn = p_first;
    for (int t = first; t + step < nT; t += step) {  // (no division in front of the rows, as in the kernel)
      pn += pstep;
#pragma unroll
      for (int i = 0; i < 4; ++i) fold ^= fold16(T.ka[i]) ^ fold16(T.kb[i]);   // the K half is consumed ...
      ra = W.row_of(pn + n, sAn);
      rb = W.row_of(pn + 16 + n, sBn);
      issue_k_rows<uint32_t, WIDE>(T, R, ra, rb);                              // ... and refilled,
      sAn = W.sel_at_nonempty(pn + pstep + n);
      sBn = W.sel_at_nonempty(pn + pstep + 16 + n);
#pragma unroll
      for (int i = 0; i < 8; ++i) fold ^= fold16(T.v[i]);                      // then the V half
      issue_v_rows<uint32_t, WIDE>(T, R, ra, rb);
    }
    if (first < nT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) fold ^= fold16(T.ka[i]) ^ fold16(T.kb[i]);
#pragma unroll
      for (int i = 0; i < 8; ++i) fold ^= fold16(T.v[i]);
    }
  }
  if (TAIL != 0) {
    f32x4 acc[8];
    const float v = (float)(fold & 0xffu);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = f32x4{v, v, v, v};
    __shared__ __align__(16) float s_red[kWaves][WIDE ? 8 : 16][kHeadDim];
    finish_wg<false, WIDE ? 1 : 2, TAIL == 2>(wg_out_of(a, bh), head0, G, slot, acc, 0.f, 1.f, &s_red[0][0][0], (WIDE ? 8 : 16) * kHeadDim);
  } else {
    fold ^= __shfl_xor(fold, 32);
    if (lane == 0) reinterpret_cast<uint32_t*>(a.part)[((head0 * a.slot_cap + slot) * kPartStride) + w] = fold;
  }
  report_guard(a.guard, W.bad);
}

// The leading arguments of the gather kernel, its skeleton and the compact kernel, and their grid (fast_cell).
static uint32_t fast_shape(const AttnArgs& a, int B) {
  const uint32_t meta = (uint32_t)a.Hkv | (a.ms == 4 ? 2u << 16 : 0u) | (a.is_slow != nullptr ? 1u << 20 : 0u);
  if (a.handover == 0) return meta;
  const uint32_t full = a.handover == 2 ? 8u << 28 : 0u;
  if (a.Hkv >= 8) return meta | 31u << 23 | full;
  const uint32_t lg = a.Hkv == 4 ? 2u : a.Hkv == 2 ? 1u : 0u;
  return meta | (3u - lg) << 21 | lg << 23 | (B * a.Hkv < 8 ? (uint32_t)(B * a.Hkv) << 28 : full);
}
static dim3 fast_grid(const AttnArgs& a, int B, int n_slots) {
  if (a.handover == 0) return dim3(n_slots, a.Hkv, B);
  const int row = a.Hkv >= 8 ? a.Hkv : 8;
  return dim3(row + (a.handover == 2 ? 1 : 0), n_slots, (B * a.Hkv + row - 1) / row);
}
static const uint8_t* gather_flags(const AttnArgs& a) {  // (a readable byte in any case)
  return a.is_slow != nullptr ? a.is_slow : reinterpret_cast<const uint8_t*>(a.ctx_len);
}
hipError_t launch_attn_gather_floor(const AttnArgs& a, int B, int n_slots, int tail, int burst, int tpw, int depth, hipStream_t s) {
  const dim3 grid = fast_grid(a, B, n_slots);
  const size_t lds = burst ? (size_t)tpw * 16 * 64 * sizeof(uint4) : 0;
#define SFI_FLOOR(WIDE, TAIL, BURST)                                                                                   \
  do {                                                                                                                 \
    if (lds > 0 && hipFuncSetAttribute(reinterpret_cast<const void*>(&attn_gather_floor_kernel<WIDE, TAIL, BURST>),   \
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)            \
      return hipGetLastError();                                                                                        \
    hipLaunchKernelGGL((attn_gather_floor_kernel<WIDE, TAIL, BURST>), grid, dim3(kAttnThreads), lds, s, a.sel_idx, a.n_sel,   \
                       a.ctx_len, a.recent_start, gather_flags(a), (uint32_t)a.sel_stride, fast_shape(a, B), a.n_sink,        \
                       a.n_split, a, tpw, depth);                                                                              \
  } while (0)
  const bool wide = a.G <= 8;
  if (tail) {  // (never with a burst)
    if (wide && a.handover != 0) SFI_FLOOR(true, 2, false);
    else if (wide) SFI_FLOOR(true, 1, false);
    else if (a.handover != 0) SFI_FLOOR(false, 2, false);
    else SFI_FLOOR(false, 1, false);
  } else if (wide && burst) SFI_FLOOR(true, 0, true);
  else if (wide) SFI_FLOOR(true, 0, false);
  else if (burst) SFI_FLOOR(false, 0, true);
  else SFI_FLOOR(false, 0, false);
#undef SFI_FLOOR
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Memory skeleton of the dense kernel -- a measurement aid, not part of the path: the dense launch's grid and
// tile dealing (tiles first, first + step, ... of the prefix per wave, two tile buffers in flight, K half and V
// half of a buffer refilled separately; tile t starts at row n_sink + 32 t as the kernel's tiles of J do), nontemporal
// 16-byte loads, nothing computed: what arrives is folded
// into one word per wave.  WIDE: K rows requested as whole 128-byte lines (the gather kernels' layout) instead
// of the four 64-byte pieces the dense kernel's operand layout asks for.  No logits are written.
// The eight loads of a half go out back to back, as the kernel issues them (left to itself the compiler refills
// register by register as the fold frees them, and that order of requests is 10 % slower).  idle_units > 0: the wave
// sleeps idle_units x 64 cycles where the kernel has its two blocks of arithmetic (after the K half and after the V
// half of every tile), to show what time between the waits costs when the memory side is the same.
// writer > 0: the workgroup has a fifth wave that does nothing but store what the kernel would expose (G x 128 bytes
// per tile, the kernel's addresses; writer == 2: always the same 2 KB of them), at about the readers' pace, while the
// four waves read: what store instructions cost a compute unit that is streaming rows.
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ void idle(int units) {
  for (int i = 0; i < units; ++i) __builtin_amdgcn_s_sleep(1);
}
template <bool WIDE>
__global__ __launch_bounds__(kAttnThreads + 64, 1) void attn_dense_floor_kernel(const AttnArgs a, int idle_units, int writer) {
  const int slot = blockIdx.y, h = blockIdx.x, b = blockIdx.z;
  const int tid = threadIdx.x;
  const int lane = tid & 63, w = tid >> 6;
  const int jg = lane >> 4, n = lane & 15;
  if (w == kWaves) {  // the writer wave (only launched with writer > 0)
    int bad0 = 0;
    const int L0 = guarded_len(a.ctx_len[b * a.ms], a.len_cap, bad0);
    const int nT0 = (L0 + kTile - 1) / kTile;
    const int step0 = a.n_split * kWaves;
    float* lg = a.logits + (int64_t)(b * a.Hkv + h) * a.G * a.ld_pos;
    const int tile_floats = a.G * kTile;
    const int k_max = slot * kWaves < nT0 ? (nT0 - slot * kWaves + step0 - 1) / step0 : 0;
    for (int k = 0; k < k_max; ++k) {
      __builtin_amdgcn_s_sleep(90);  // 5760 cycles: a little less than the four waves take per tile
      for (int ww = 0; ww < kWaves; ++ww) {
        const int t = slot * kWaves + ww + k * step0;
        if (t < a.max_tiles && lane * 4 < tile_floats)
          *reinterpret_cast<float4*>(lg + (int64_t)(writer == 2 ? ww : t) * tile_floats + lane * 4) = make_float4((float)lane, 0.f, 0.f, 0.f);
      }
    }
    return;
  }
  Rows R;
  R.Kb = reinterpret_cast<const char*>(a.K + b * a.k_sb + h * a.k_sh);
  R.Vb = reinterpret_cast<const char*>(a.V + b * a.v_sb + h * a.v_sh);
  R.k_st = (uint32_t)a.k_st * 2u;
  R.v_st = (uint32_t)a.v_st * 2u;
  R.k_lane = k_lane_of<WIDE>(jg, n);
  R.v_lane = n * 16;
  R.jg = jg;
  R.n = n;
  const int first = slot * kWaves + w, step = a.n_split * kWaves;
  Tile T, T2;
  issue_affine<WIDE>(T, R, a.n_sink + first * kTile, a.row_cap);  // before ctx_len arrives, as the kernel does
  issue_affine<WIDE>(T2, R, a.n_sink + (first + step) * kTile, a.row_cap);
  int bad = 0;
  const int L = guarded_len(a.ctx_len[b * a.ms], a.len_cap, bad);
  const int r_last = max(L, 1) - 1;
  const int nT = (L + kTile - 1) / kTile;
  const int K = first < nT ? (nT - first + step - 1) / step : 0;
  uint32_t fold = 0u;
  auto use = [&](Tile& B, int k) {
    const int t_next = first + (k + 2) * step;
#pragma unroll
    for (int i = 0; i < 4; ++i) fold ^= fold16(B.ka[i]) ^ fold16(B.kb[i]);
    __builtin_amdgcn_sched_barrier(0);
    idle(idle_units);
    __builtin_amdgcn_sched_barrier(0);
    issue_k_affine<WIDE>(B, R, a.n_sink + t_next * kTile, r_last);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 8; ++i) fold ^= fold16(B.v[i]);
    __builtin_amdgcn_sched_barrier(0);
    idle(idle_units);
    __builtin_amdgcn_sched_barrier(0);
    issue_v_affine<WIDE>(B, R, a.n_sink + t_next * kTile, r_last);
    __builtin_amdgcn_sched_barrier(0);
  };
  int k = 0;
  for (; k + 1 < K; k += 2) {
    use(T, k);
    use(T2, k + 1);
  }
  if (k < K) use(T, k);
#pragma unroll
  for (int i = 0; i < 4; ++i) fold ^= fold16(T.ka[i]) ^ fold16(T.kb[i]) ^ fold16(T2.ka[i]) ^ fold16(T2.kb[i]);  // the refills past the end
#pragma unroll
  for (int i = 0; i < 8; ++i) fold ^= fold16(T.v[i]) ^ fold16(T2.v[i]);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) fold ^= __shfl_xor(fold, d);
  const int64_t head0 = (int64_t)b * a.Hq + h * a.G;
  if (lane == 0) reinterpret_cast<uint32_t*>(a.part)[((head0 * kSlotCap + slot) * kPartStride) + w] = fold;
}
hipError_t launch_attn_dense_floor(const AttnArgs& a, int B, int n_slots, int wide, int idle_units, int writer, hipStream_t s) {
  const dim3 grid(a.Hkv, n_slots, B);
  const dim3 block(writer != 0 ? kAttnThreads + 64 : kAttnThreads);
  if (wide) hipLaunchKernelGGL(attn_dense_floor_kernel<true>, grid, block, 0, s, a, idle_units, writer);
  else hipLaunchKernelGGL(attn_dense_floor_kernel<false>, grid, block, 0, s, a, idle_units, writer);
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// compact kernel: the fast step over the two-segment layout (Sec. "Memory-coalesced Kernel Design
// and Selector Maintenance"): sink ++ selected rows from the compact buffers the Reorg kernel filled,
// the recent window in place from the cache.  Both segments are runs of consecutive rows, so no
// index is read: a wave's first tile is on its way before any scalar of the step has arrived.
// Tiles never straddle the two segments: the compact segment ends with a ragged tile of its own.
// ------------------------------------------------------------------------------------------------
// What the first tile's rows need arrives in registers, the flag of a ragged step is looked at behind their requests, and the last
// tile is not refilled: us a layer, 8 KV heads, at device scope 15.31 -> 15.15 (12 x 5003..30011 rows, budget 1024), 11.92 -> 11.75 (4 x 32768, 2048),
// 10.49 -> 9.78 (131072, 4096); records through the L2 14.92, 11.63, 9.66.
template <bool PAGED, bool WIDE, bool LOCAL>  // PAGED: the recent window is read from a paged cache (the compact buffers are always flat)
__device__ __forceinline__ void compact_body(const FastCell& cell, const uint16_t* Kc, const uint16_t* Vc, const uint8_t* is_slow_p,
                                             const int64_t c_sb, const int64_t c_sh, const uint32_t shape, const int c_rows, const int n_split,
                                             const AttnArgs& a, float* lds) {
  const int slot = cell.slot, h = cell.h, b = cell.b;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int jg = lane >> 4, n = lane & 15;
  const bool flagged = ((shape >> 20) & 1u) != 0u;
  const int first = slot * kWaves + w, step = n_split * kWaves;

  Rows Rc;  // compact segment
  Rc.Kb = reinterpret_cast<const char*>(Kc + b * c_sb + h * c_sh);
  Rc.Vb = reinterpret_cast<const char*>(Vc + b * c_sb + h * c_sh);
  Rc.k_st = Rc.v_st = kHeadDim * 2u;
  Rc.k_lane = k_lane_of<WIDE>(jg, n);
  Rc.v_lane = n * 16;
  Rc.jg = jg;
  Rc.n = n;
  Tile T;
  const bool spec = first * kTile < c_rows;  // almost every wave's tile lies in the compact segment
  if (spec) issue_affine<WIDE>(T, Rc, first * kTile, c_rows - 1);
  const int slow = is_slow_p[flagged ? (uint32_t)b << (2u * ((shape >> 16) & 15u)) : 0u];  // (a readable byte in any case)
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::"s"(a.q), "s"(a.K), "s"(a.V), "s"(a.k_sb), "s"(a.k_sh), "s"(a.k_st), "s"(a.v_sb), "s"(a.v_sh), "s"(a.v_st), "s"(a.ctx_len),
               "s"(a.n_sel), "s"(a.recent_start), "s"(a.ms), "s"(a.Hq), "s"(a.Hkv), "s"(a.G), "s"(a.n_sink), "s"(a.len_cap), "s"(a.sel_stride));
  const int G = a.G;
  const int bh = b * a.Hkv + h;
  const int64_t head0 = (int64_t)b * a.Hq + h * G;
  Rows R = Rc;  // recent segment, in the cache
  R.Kb = reinterpret_cast<const char*>(a.K + b * a.k_sb + h * a.k_sh);
  R.Vb = reinterpret_cast<const char*>(a.V + b * a.v_sb + h * a.v_sh);
  R.k_st = (uint32_t)a.k_st * 2u;
  R.v_st = (uint32_t)a.v_st * 2u;

  bf16x8 qreg[4];
  load_q<WIDE>(qreg, a.q, head0, G, jg, n);
  int bad = 0;
  const int L_in = a.ctx_len[b * a.ms], nSel0 = a.n_sel[bh], rs_in = a.recent_start[b * a.ms];  // one round trip for the three
  if (flagged && __builtin_amdgcn_readfirstlane(slow) != 0) return;
  const int L = guarded_len(L_in, a.len_cap, bad);
  const int nSel = min(max(nSel0, 0), (int)a.sel_stride);
  bad |= nSel != nSel0 ? kGuardNSel : 0;
  const int nS = min(a.n_sink, L);
  // A context that still lies inside the sink range has nothing selected, and the rows appended since
  // the reorganisation are sink rows the compact buffers do not hold: all of it is read in place.
  const bool all_sink = L <= a.n_sink;
  const int rs = all_sink ? 0 : min(max(rs_in, nS), L);
  const int Nc = all_sink ? 0 : a.n_sink + nSel;  // compact rows in use
  const int Tc = (Nc + kTile - 1) / kTile;
  const int Nr = L - rs;
  const int nT = Tc + (Nr + kTile - 1) / kTile;

  float m_run = kNeg, l_run = 0.f;
  f32x4 acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Tile t < Tc is rows 32 t .. of the compact segment, tile t >= Tc rows rs + 32 (t - Tc) .. of the cache
  // (clamped to L - 1).  The branch is wave-uniform and both sides issue the same number of loads.
  int pra_n = 0, prb_n = 0;  // PAGED: physical rows of the recent tile whose K half was issued last
  auto issue_k_tile = [&](int t) {
    if (t < Tc) {
      issue_k_affine<WIDE>(T, Rc, t * kTile, c_rows - 1);
    } else if (PAGED) {
      const Pages P = pages_of(a, b, L);
      const int ra = min(rs + (t - Tc) * kTile + n, L - 1), rb = min(rs + (t - Tc) * kTile + 16 + n, L - 1);
      pra_n = P.phys(ra, P.page_of(ra), bad);
      prb_n = P.phys(rb, P.page_of(rb), bad);
      issue_k_rows<uint64_t, WIDE>(T, R, pra_n, prb_n);
    } else {
      issue_k_affine<WIDE>(T, R, rs + (t - Tc) * kTile, L - 1);
    }
  };
  auto issue_v_tile = [&](int t) {
    if (t < Tc) issue_v_affine<WIDE>(T, Rc, t * kTile, c_rows - 1);
    else if (PAGED) issue_v_rows<uint64_t, WIDE>(T, R, pra_n, prb_n);
    else issue_v_affine<WIDE>(T, R, rs + (t - Tc) * kTile, L - 1);
  };
  const int K = first < nT ? (nT - first + step - 1) / step : 0;
  if (K > 0 && !(spec && first < Tc)) {  // the first tile is not the compact tile requested up front
    issue_k_tile(first);
    issue_v_tile(first);
  }
  // the dense kernel's loop: K half refilled after S^T, V half after P V (next < 0: not refilled)
  auto tile_step = [&](int t, int next) {
    const int p0 = (t < Tc ? t : t - Tc) * kTile;
    const int N = t < Tc ? Nc : Nr;
    float y[8];
    qk_phase<WIDE>(T, qreg, a.scale_log2, y);
    if (next >= 0) issue_k_tile(next);
    if (p0 + kTile > N) mask_tail<WIDE>(T, y, jg, p0, N);
    bf16x8 a_hi, a_lo;
    softmax_phase(y, acc, m_run, l_run, jg, a_hi, a_lo);
    pv_phase(T, a_hi, a_lo, acc);
    if (next >= 0) issue_v_tile(next);
  };
  // (the last tile apart: no rows are requested for a tile that does not exist)
  if (K > 0) {
    int t = first;
    for (int k = 1; k < K; ++k, t += step) tile_step(t, t + step);
    tile_step(t, -1);
  }
  const WgOut o = wg_out_of(a, bh);
  if (finish_wg<false, WIDE ? 1 : 2, LOCAL>(o, head0, G, slot, acc, m_run, rows_sum(l_run), lds, (WIDE ? 8 : 16) * kHeadDim)) {
    m_run = kNeg;
    l_run = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int t = 0; t < nT; ++t) {
      issue_k_tile(t);
      issue_v_tile(t);
      tile_step(t, -1);
    }
    store_heads(o, head0, G, acc, l_run);
  }
  report_guard(a.guard, bad);
}
template <bool PAGED, bool WIDE, bool LOCAL>
__global__ __launch_bounds__(kAttnThreads, PAGED ? 2 : 3) void attn_compact_kernel(const uint16_t* Kc, const uint16_t* Vc, const uint8_t* is_slow_p,
                                                                                   const int64_t c_sb, const int64_t c_sh, const uint32_t shape,
                                                                                   const int c_rows, const int n_split, const AttnArgs a) {
  const FastCell cell = fast_cell<LOCAL>(shape);
  if (cell.off) return;
  __shared__ __align__(16) float s_red[kWaves * (WIDE ? 8 : 16) * kHeadDim];
  compact_body<PAGED, WIDE, LOCAL>(cell, Kc, Vc, is_slow_p, c_sb, c_sh, shape, c_rows, n_split, a, s_red);
}

// ------------------------------------------------------------------------------------------------
// The ragged step's attention in one launch: a workgroup takes a cell of the fast sequences, as in the gather or the compact
// launch, and then its share of the slow ones, as in the planned dense launch, for as many cells as there are shares.  One
// launch less, the start of the dense part and the hand-over of the fast part hide behind each other, and a workgroup whose
// cell belongs to a slow sequence begins its share at once.  (The other order gains half of that: the cell's first loads
// wait for the acknowledgement of the share's last stores.)
// Two launches / one, us a step with the Selector behind it: 12 x 5003..30011 rows, budget 1024, compact buffers, 1 slow 53.6 / 50.7, 4 slow 93.2 / 90.2; 8 x
// 20011..24571, G = 5, paged, 1 slow 48.1 / 44.6; 4 x 5515..14434, G = 8, 1 slow 38.2 / 35.4; 64 x 1000..3000, 2 KV heads, 3 slow 25.0 / 22.2, 16 slow 29.8 / 27.4.
// With more cells than shares the fast part loses the two other workgroups a unit would hold: 128 x 3000..8000 rows 128 / 136.
// ------------------------------------------------------------------------------------------------
// BALANCED (balanced_shares): the shares are cut by what a workgroup has had already (PlanCells).  (Every head has its
// workgroups with a cell in the same places: the heads' shares alternate as the cells do.)
template <bool PAGED, bool WIDE, bool COMPACT, bool BALANCED>
__global__ __launch_bounds__(kAttnThreads, 1) void attn_ragged_kernel(const int32_t* ctx_len, const uint8_t* is_slow, const int32_t* recent_start,
                                                                      const int32_t* sel_idx, const uint32_t strides, const uint32_t shape, const int B,
                                                                      const int W_max, const int n_sink, const int n_split, const float per_min,
                                                                      const int row_in, const float cell_tiles, const AttnArgs f, const AttnArgs d) {
  __shared__ __align__(16) float s_patch[kWaves * patch_floats(1, true)];
  const uint32_t id = blockIdx.x, Hkv = shape & 0xffffu;
  // the cells in the order of fast_grid: row pairs side by side, n_split slots of them, then the next row.  row_in: the pairs in a
  // row, negative (tests): which of them a workgroup has changes from slot to slot, and with it the XCD of a pair's slots.
  const uint32_t row = abs(row_in), q = id / row, z = q / (uint32_t)n_split, slot = q - z * n_split;
  const uint32_t pair = z * row + ((id - q * row) ^ (row_in < 0 ? slot & 7u : 0u));
  const FastCell cell{(int)slot, (int)(pair % Hkv), (int)(pair / Hkv), false};
  const int j = id / Hkv, h = id - (uint32_t)j * Hkv;
  PlanCells cells;
  if (BALANCED) {
    const int bc0 = min((int)(threadIdx.x & 63) * ((B + 63) / 64), B - 1);
    cells = PlanCells{n_split, (int)((shape >> 21) & 3u), cell_tiles, ctx_len[bc0 * (int)(strides & 0xffffu)], is_slow[bc0 * (int)(strides >> 16)]};
  }
  if (cell.b < B) {
    if (COMPACT) compact_body<PAGED, WIDE, true>(cell, f.Kc, f.Vc, is_slow, f.c_sb, f.c_sh, shape, f.c_rows, n_split, f, s_patch);
    else gather_body<PAGED, WIDE, true>(cell, sel_idx, f.n_sel, ctx_len, recent_start, is_slow, (uint32_t)f.sel_stride, shape, n_sink, n_split, f, s_patch);
  }
  __syncthreads();  // the cell's results in LDS have been read
  Scored sc = scored_of(s_patch);
  if (id < (uint32_t)W_max * Hkv)
    planned_body<1, PAGED, false, BALANCED>(j, h, ctx_len, is_slow, nullptr, strides, B, W_max, per_min, n_sink, d.recent, d.len_cap, d, s_patch, sc, cells);
}

// ------------------------------------------------------------------------------------------------
// Reorg (Sec. "Hiding Slow-step Overhead via Layer-wise Asynchronous Execution": Reorg_i): compact row
// i < n_sink is cache row i, compact row n_sink + i is cache row sel_idx[i], i < n_sel.  A workgroup
// moves kReorgRows compact rows of one (b, h), 16 lanes x 16 bytes per row, K and V; the indices
// are read before the list length is known, and all of a thread's row loads precede its stores.
// ------------------------------------------------------------------------------------------------
template <bool PAGED>
__global__ __launch_bounds__(kAttnThreads) void reorg_kernel(const ReorgArgs a) {
  const int chunk = blockIdx.x, h = blockIdx.y, b = blockIdx.z;
  if (a.is_slow != nullptr && a.is_slow[b * a.fs] == 0) return;
  const int bh = b * a.Hkv + h;
  const int tid = threadIdx.x;
  const int sub = tid & 15, r = tid >> 4;
  constexpr int kPass = kReorgRows / 16;
  const int32_t* sel = a.sel_idx + (int64_t)bh * a.sel_stride;
  const int sel_cap = (int)a.sel_stride - 1;
  int src[kPass];
#pragma unroll
  for (int p = 0; p < kPass; ++p) {
    const int i = chunk * kReorgRows + p * 16 + r;
    src[p] = sel_cap >= 0 ? sel[min(max(i - a.n_sink, 0), sel_cap)] : 0;
  }
  int bad = 0;
  const int L_in = a.ctx_len[b * a.ms], nSel0 = a.n_sel[bh];
  const int L = guarded_len(L_in, a.len_cap, bad);
  const int nSel = min(max(nSel0, 0), (int)a.sel_stride);
  bad |= nSel != nSel0 ? kGuardNSel : 0;
  const int nS = min(a.n_sink, L);
  const int r_hi = max(L, 1) - 1;
  const char* Kb = reinterpret_cast<const char*>(a.K + b * a.k_sb + h * a.k_sh);
  const char* Vb = reinterpret_cast<const char*>(a.V + b * a.v_sb + h * a.v_sh);
  char* Kc = reinterpret_cast<char*>(a.Kc + b * a.c_sb + h * a.c_sh);
  char* Vc = reinterpret_cast<char*>(a.Vc + b * a.c_sb + h * a.c_sh);
  uint4 kr[kPass], vr[kPass];
  bool ok[kPass];
#pragma unroll
  for (int p = 0; p < kPass; ++p) {
    const int i = chunk * kReorgRows + p * 16 + r;
    ok[p] = i < nS || (i >= a.n_sink && i < a.n_sink + nSel);
    int row = i < a.n_sink ? i : src[p];
    if (ok[p]) {  // a stored index outside the context reads as the context's last row (as in the gather kernels)
      const int rc = (int)min((uint32_t)row, (uint32_t)r_hi);
      bad |= rc != row ? kGuardSelIdx : 0;
      row = rc;
    }
    if (PAGED && ok[p]) {
      const int32_t* tbl = a.table + (int64_t)b * a.table_stride;
      const int page = tbl[row >> a.page_lg];
      const int pc = min(max(page, 0), a.n_blocks - 1);
      bad |= pc != page ? kGuardBlock : 0;
      row = pc * a.page_rpb + (row & ((1 << a.page_lg) - 1));
    }
    if (ok[p]) {
      typedef typename RowOff<PAGED>::type OffT;
      kr[p] = load_row16(Kb, (OffT)((OffT)(uint32_t)row * ((uint32_t)a.k_st * 2u) + sub * 16));
      vr[p] = load_row16(Vb, (OffT)((OffT)(uint32_t)row * ((uint32_t)a.v_st * 2u) + sub * 16));
    }
  }
#pragma unroll
  for (int p = 0; p < kPass; ++p) {
    const int i = chunk * kReorgRows + p * 16 + r;
    if (ok[p]) {
      *reinterpret_cast<uint4*>(Kc + (int64_t)i * (kHeadDim * 2) + sub * 16) = kr[p];
      *reinterpret_cast<uint4*>(Vc + (int64_t)i * (kHeadDim * 2) + sub * 16) = vr[p];
    }
  }
  report_guard(a.guard, bad);
}

// Stand-alone merge: one workgroup per (sequence, query head).
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(const MergeArgs a) {
  const int bg = blockIdx.x;
  const int b = bg / a.Hq;
  int n_slots;
  if (a.mode == 2 && a.slots_fast == 0 && a.is_slow[b * a.fs] == 0) return;  // fast sequences wrote their output themselves
  if (a.mode == 0) n_slots = a.slots_slow;
  else if (a.mode == 1) n_slots = a.slots_fast;
  else n_slots = a.is_slow[b * a.fs] ? a.slots_slow : a.slots_fast;
  if (a.mode == 0 && a.seq_rec != nullptr) n_slots = a.seq_rec[b];
  const bool dense = a.mode == 0 || (a.mode == 2 && a.is_slow[b * a.fs]);
  merge_records(a.part, a.out, bg, n_slots, dense ? a.jstat : nullptr, a.G, a.alpha, a.out_bf16 != 0);
}

__global__ void advance_kernel(int32_t* ctx_len, int32_t* recent_start, int B, int n_sink, int recent) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) {
    const int L = ctx_len[b] + 1;
    ctx_len[b] = L;
    recent_start[b] = max(n_sink, L - recent);
  }
}

__global__ void trigger_kernel(const int32_t* last_token, const uint32_t* bitmap, int vocab, int t_max, int32_t* since_slow,
                               uint8_t* is_slow, int B) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) {
    const int tok = last_token[b];
    const int c = since_slow[b];
    const bool hit = tok >= 0 && tok < vocab && ((bitmap[tok >> 5] >> (tok & 31)) & 1u) != 0u;
    const bool slow = hit || c >= t_max;
    is_slow[b] = slow ? 1 : 0;
    since_slow[b] = slow ? 0 : c + 1;
  }
}

// The packed per-step descriptor (Sec. "Memory-coalesced Kernel Design and Selector Maintenance": built once per
// decoding step, read by every kernel of the step): state update and trigger decision of every sequence in one launch.
__global__ void step_begin_kernel(sfi_step_desc* desc, const int32_t* last_token, const uint32_t* bitmap, int vocab, int t_max,
                                  int advance, int B, int n_sink, int recent) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) {
    sfi_step_desc d = desc[b];
    if (advance) d.ctx_len += 1;
    d.recent_start = max(n_sink, d.ctx_len - recent);
    const int tok = last_token != nullptr ? last_token[b] : -1;
    const bool hit = bitmap != nullptr && tok >= 0 && tok < vocab && ((bitmap[tok >> 5] >> (tok & 31)) & 1u) != 0u;
    const bool slow = hit || d.since_slow >= t_max;
    d.is_slow = slow ? 1 : 0;
    d.since_slow = slow ? 0 : d.since_slow + 1;
    desc[b] = d;
  }
}
hipError_t launch_step_begin(sfi_step_desc* desc, const int32_t* last_token, const uint32_t* bitmap, int vocab, int t_max,
                             int advance, int B, int n_sink, int recent, hipStream_t s) {
  hipLaunchKernelGGL(step_begin_kernel, dim3((B + 63) / 64), dim3(64), 0, s, desc, last_token, bitmap, vocab, t_max, advance, B,
                     n_sink, recent);
  return hipGetLastError();
}

hipError_t launch_trigger(const int32_t* last_token, const uint32_t* bitmap, int vocab, int t_max, int32_t* since_slow,
                          uint8_t* is_slow, int B, hipStream_t s) {
  hipLaunchKernelGGL(trigger_kernel, dim3((B + 63) / 64), dim3(64), 0, s, last_token, bitmap, vocab, t_max, since_slow,
                     is_slow, B);
  return hipGetLastError();
}

template <bool PAGED>
static void launch_dense_t(const AttnArgs& a, dim3 grid, hipStream_t s) {
  if (a.plan_batch > 0) {
    const dim3 pgrid(a.Hkv, std::max(a.plan_wgs, a.plan_even * a.plan_batch));
    const uint32_t strides = (uint32_t)a.ms | (uint32_t)a.fs << 16;
#define SFI_PLANNED(EXPOSE)                                                                                             \
  hipLaunchKernelGGL((attn_dense_planned_kernel<EXPOSE, PAGED>), pgrid, dim3(kAttnThreads), 0, s, a.ctx_len, a.is_slow, \
                     a.q_len, strides, a.plan_batch, a.plan_wgs, 1.0f / (float)a.plan_min, a.n_sink, a.recent, a.len_cap, a)
    if (a.logits == nullptr) SFI_PLANNED(0);
    else if (a.with_knorm && a.met != nullptr) SFI_PLANNED(4);
    else if (a.with_knorm) SFI_PLANNED(2);
    else if (a.met != nullptr) SFI_PLANNED(3);
    else SFI_PLANNED(1);
#undef SFI_PLANNED
    return;
  }
  if constexpr (!PAGED) {
    if (a.dense_wide && a.G <= 8 && !a.with_knorm) {
      if (a.logits != nullptr && a.big_stash) hipLaunchKernelGGL((attn_dense_kernel<1, false, true, true>), grid, dim3(kAttnThreads), 0, s, a);
      else if (a.logits != nullptr) hipLaunchKernelGGL((attn_dense_kernel<1, false, false, true>), grid, dim3(kAttnThreads), 0, s, a);
      else hipLaunchKernelGGL((attn_dense_kernel<0, false, false, true>), grid, dim3(kAttnThreads), 0, s, a);
      return;
    }
  }
  if (a.met != nullptr && a.with_knorm)
    hipLaunchKernelGGL((attn_dense_kernel<4, PAGED, true>), grid, dim3(kAttnThreads), 0, s, a);
  else if (a.met != nullptr)
    hipLaunchKernelGGL((attn_dense_kernel<3, PAGED, true>), grid, dim3(kAttnThreads), 0, s, a);
  else if (a.logits != nullptr && a.with_knorm && a.big_stash)
    hipLaunchKernelGGL((attn_dense_kernel<2, PAGED, true>), grid, dim3(kAttnThreads), 0, s, a);
  else if (a.logits != nullptr && a.with_knorm)
    hipLaunchKernelGGL((attn_dense_kernel<2, PAGED>), grid, dim3(kAttnThreads), 0, s, a);
  else if (a.logits != nullptr && a.big_stash)
    hipLaunchKernelGGL((attn_dense_kernel<1, PAGED, true>), grid, dim3(kAttnThreads), 0, s, a);
  else if (a.logits != nullptr)
    hipLaunchKernelGGL((attn_dense_kernel<1, PAGED>), grid, dim3(kAttnThreads), 0, s, a);
  else {
    if constexpr (PAGED) {
      if (a.big_stash) {  // (no stash without logits: one workgroup per unit is what is meant, and its registers)
        hipLaunchKernelGGL((attn_dense_kernel<0, true, true>), grid, dim3(kAttnThreads), 0, s, a);
        return;
      }
    }
    hipLaunchKernelGGL((attn_dense_kernel<0, PAGED>), grid, dim3(kAttnThreads), 0, s, a);
  }
}
hipError_t launch_attn_dense(const AttnArgs& a, int B, int n_slots, hipStream_t s) {
  const dim3 grid(a.Hkv, n_slots, B);
  if (a.table != nullptr) launch_dense_t<true>(a, grid, s);
  else launch_dense_t<false>(a, grid, s);
  return hipGetLastError();
}
hipError_t launch_attn_ragged(const AttnArgs& d, const AttnArgs& f, bool balanced, hipStream_t s) {
  const int B = d.plan_batch;
  const int row = f.handover == 0 || f.Hkv >= 8 ? f.Hkv : 8;  // as fast_grid
  const int cells = (B * f.Hkv + row - 1) / row * row * f.n_split;
  const dim3 grid(std::max(d.plan_wgs * d.Hkv, cells)), block(kAttnThreads);
  const uint32_t strides = (uint32_t)d.ms | (uint32_t)d.fs << 16;
  // A cell's tile takes less than the list's, whose logits are exposed.  (0.8 / 0.9, us a step: 32 x 8192 rows, half slow, 125.1 / 131.2; 16 x
  // 16384..49152, half slow, 219.5 / 222.2; 16 x 16384..65536, budget 1024, a quarter slow, 148.5 / 146.0.)
  const float cell_tiles = 0.8f * std::min((float)f.n_sink + (float)f.sel_stride + (float)f.recent, (float)d.len_cap) / (float)(kTile * f.n_split);
#define SFI_RAGGED(PAGED, WIDE, COMPACT, BALANCED)                                                                                                 \
  hipLaunchKernelGGL((attn_ragged_kernel<PAGED, WIDE, COMPACT, BALANCED>), grid, block, 0, s, d.ctx_len, d.is_slow, f.recent_start, f.sel_idx,     \
                     strides, fast_shape(f, B), B, d.plan_wgs, d.n_sink, f.n_split, 1.0f / (float)d.plan_min, f.handover == 2 ? -row : row,       \
                     cell_tiles, f, d)
#define SFI_RAGGED_C(PAGED, COMPACT)                                   \
  do {                                                                 \
    if (f.G <= 8 && balanced) SFI_RAGGED(PAGED, true, COMPACT, true);  \
    else if (f.G <= 8) SFI_RAGGED(PAGED, true, COMPACT, false);        \
    else if (balanced) SFI_RAGGED(PAGED, false, COMPACT, true);        \
    else SFI_RAGGED(PAGED, false, COMPACT, false);                     \
  } while (0)
  if (d.table != nullptr && f.Kc != nullptr) SFI_RAGGED_C(true, true);
  else if (d.table != nullptr) SFI_RAGGED_C(true, false);
  else if (f.Kc != nullptr) SFI_RAGGED_C(false, true);
  else SFI_RAGGED_C(false, false);
#undef SFI_RAGGED_C
#undef SFI_RAGGED
  return hipGetLastError();
}
hipError_t launch_attn_compact(const AttnArgs& a, int B, int n_slots, hipStream_t s) {
  const dim3 grid = fast_grid(a, B, n_slots), block(kAttnThreads);
#define SFI_COMPACT(PAGED, WIDE)                                                                                                            \
  do {                                                                                                                                      \
    if (a.handover != 0)                                                                                                                    \
      hipLaunchKernelGGL((attn_compact_kernel<PAGED, WIDE, true>), grid, block, 0, s, a.Kc, a.Vc, gather_flags(a), a.c_sb, a.c_sh,           \
                         fast_shape(a, B), a.c_rows, a.n_split, a);                                                                          \
    else                                                                                                                                    \
      hipLaunchKernelGGL((attn_compact_kernel<PAGED, WIDE, false>), grid, block, 0, s, a.Kc, a.Vc, gather_flags(a), a.c_sb, a.c_sh,          \
                         fast_shape(a, B), a.c_rows, a.n_split, a);                                                                          \
  } while (0)
  if (a.G <= 8) {
    if (a.table != nullptr) SFI_COMPACT(true, true);
    else SFI_COMPACT(false, true);
  } else {
    if (a.table != nullptr) SFI_COMPACT(true, false);
    else SFI_COMPACT(false, false);
  }
#undef SFI_COMPACT
  return hipGetLastError();
}
hipError_t launch_reorg(const ReorgArgs& a, int B, int rows, hipStream_t s) {
  const dim3 grid((rows + kReorgRows - 1) / kReorgRows, a.Hkv, B);
  if (a.table != nullptr) hipLaunchKernelGGL(reorg_kernel<true>, grid, dim3(kAttnThreads), 0, s, a);
  else hipLaunchKernelGGL(reorg_kernel<false>, grid, dim3(kAttnThreads), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_attn_gather(const AttnArgs& a, int B, int n_slots, hipStream_t s) {
  const dim3 grid = fast_grid(a, B, n_slots), block(kAttnThreads);
#define SFI_GATHER(PAGED, WIDE)                                                                                             \
  do {                                                                                                                      \
    if (a.handover != 0)                                                                                                    \
      hipLaunchKernelGGL((attn_gather_kernel<PAGED, WIDE, true>), grid, block, 0, s, a.sel_idx, a.n_sel, a.ctx_len,         \
                         a.recent_start, gather_flags(a), (uint32_t)a.sel_stride, fast_shape(a, B), a.n_sink, a.n_split, a); \
    else                                                                                                                    \
      hipLaunchKernelGGL((attn_gather_kernel<PAGED, WIDE, false>), grid, block, 0, s, a.sel_idx, a.n_sel, a.ctx_len,        \
                         a.recent_start, gather_flags(a), (uint32_t)a.sel_stride, fast_shape(a, B), a.n_sink, a.n_split, a); \
  } while (0)
  if (a.G <= 8) {
    if (a.table != nullptr) SFI_GATHER(true, true);
    else SFI_GATHER(false, true);
  } else {
    if (a.table != nullptr) SFI_GATHER(true, false);
    else SFI_GATHER(false, false);
  }
#undef SFI_GATHER
  return hipGetLastError();
}
hipError_t launch_merge(const MergeArgs& a, int B, hipStream_t s) {
  hipLaunchKernelGGL(merge_kernel, dim3(B * a.Hq), dim3(kMergeThreads), 0, s, a);
  return hipGetLastError();
}
hipError_t launch_advance(int32_t* ctx_len, int32_t* recent_start, int B, int n_sink, int recent, hipStream_t s) {
  hipLaunchKernelGGL(advance_kernel, dim3((B + 63) / 64), dim3(64), 0, s, ctx_len, recent_start, B, n_sink, recent);
  return hipGetLastError();
}

}  // namespace sfi
