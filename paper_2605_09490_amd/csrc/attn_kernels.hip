// Decode attention over the tiered KV cache, with cumulative-score emission (Eq. 1, Eq. 2-3 of the paper).
//
//   attn_tiered : grid (S, Hkv, B), one workgroup per compute unit.  The per-sequence lists F (T0 u T1 rows at full
//                 precision, ascending position) and Q (T2 rows, int8 / int4 codes) are cut into tiles of 32 or 64
//                 entries; T3 positions are in neither list.  The S * NW waves of a (sequence, kv head) pair are divided
//                 between the two lists so that the longest wave is shortest, and every wave walks its tiles with a stride,
//                 on its own, with no workgroup barrier until the end.
//                 Rows never pass through registers on their way in: every lane fetches 16-byte (4-byte for short
//                 code rows) pieces straight into the wave's LDS tile buffer (buffer_load ... lds).  The one buffer
//                 holds the K rows of a tile, then its V rows, then the next tile's K rows: as soon as a piece has
//                 been read, the bytes it occupied are refilled with the pieces due next, so a wave keeps about a
//                 tile's worth of rows in flight while it computes; waits are vmcnt counts derived from the fixed
//                 issue order of one tile period.
//                   K rows  - 8 lanes per row; the G logits of a row are reduced over its 8 lanes by DPP and kept
//                             by the lane whose index equals the entry's index in the tile;
//                   softmax - online, one entry per lane (exact tile maximum, exp2, running m and l);
//                   V rows  - D/EV lanes per row, probabilities broadcast from LDS, per-lane fp32 output slices.
//                 The waves of a workgroup are merged through LDS into one split partial (m, l, o[G][D]); the
//                 logits go to a scratch array.  16-bit rows of 256 bytes under four and more heads: the same launch with
//                 its waves on the matrix cores, as in attn_step.
//   attn_step   : a whole decode step's layers (or a single call over many pairs), one workgroup per (layer, sequence, kv
//                 head) pair, on the matrix cores (one or two heads a group over short lists: on the vector ALUs): the
//                 logits stay in the LDS, the workgroup writes its output itself and one float per row (the weights summed
//                 over the group) for step_scores / call_scores.
//   attn_finish : grid (64-entry tiles + Hq, B).  Every workgroup first merges the (m, l) of all splits of its sequence
//                 into the global (m, 1/l) of every query head.  Tile workgroups then turn the stored logits
//                 into softmax weights, summed over all query heads in a fixed order, into score[b, pos]; the
//                 Hq remaining workgroups merge the split outputs of one query head each into out[b, hq].
//   attn_tiered_mc : the same launch for a chunk of query tokens (tkv_attend_and_score_chunk, 16-bit rows).  The
//                 tokens ride as extra columns beside the G heads of the group (up to 32 columns per workgroup, as many
//                 groups of them as there are along grid z): per 8 KB tile a (rows x D) by (D x columns) product and its
//                 transpose-side twin for the output, which is a dense contraction and runs on the matrix cores
//                 (16x16x32 instructions; code rows widened to 16-bit values in LDS first).  Up to 32 columns and 16
//                 tokens: the logits are written and attn_finish_chunk makes scores and outputs of them.  Beyond, none
//                 are: attn_chunk_scores has the products once more, adds the weights to the scores and merges the
//                 outputs.  binary32 rows: one set of attn_tiered's workgroups per token, and attn_finish_chunk.
// The tile boundaries, the wave assignment and the fp32 summation order depend only on the lists' logical order and
// lengths, never on whether a row lives in the HBM pool or the staging buffer (both are one slot space), which is
// what makes T1 placement bit-invisible (Prop. 1).
#include <hip/hip_ext.h>

#include <algorithm>
#include <utility>

#include "tkv_internal.h"

namespace tkv {

typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) char lds_char;

constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;
constexpr int TB = TOK_PER_BLOCK;
static_assert(TB == 64, "a tile is one list entry per lane");

enum Mode : int { F_BF16 = 0, F_F32 = 1, Q_INT8 = 2, Q_INT4 = 3, F_F16 = 4 };
// type of K, V and q as a template argument: binary32, bfloat16, binary16
constexpr int KT_F32 = 0, KT_BF16 = 1, KT_F16 = 2;

template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
// f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>): loop indices usable as immediates
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// at most N vector-memory operations of this wave still outstanding (they complete in issue order)
template <int N>
__device__ __forceinline__ void wait_vm() {
  constexpr int n = N > 63 ? 63 : (N < 0 ? 0 : N);
  __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | 0x0F70);
}

// ---- LDS accesses the compiler's wait insertion does not see ------------------------------------------------
// A compiler-visible LDS load issued while direct-to-LDS loads are outstanding is preceded by a wait for all of
// them, which would serialise the pipeline; the waits for these are placed by hand (lds_fence).
template <int OFF>
__device__ __forceinline__ u32x4 lds_rd128(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
template <int OFF>
__device__ __forceinline__ u32x2 lds_rd64(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF>
__device__ __forceinline__ uint32_t lds_rd32(uint32_t addr) {
  uint32_t v;
  asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
// Transposing read: within every 16 lanes, the 4 lanes 4j .. 4j+3 point at 4 x 8 bytes that together are 16
// consecutive 16-bit elements of matrix row j (j < 4); lane i of the 16 receives element i of rows 0..3.
template <int OFF>
__device__ __forceinline__ u32x2 lds_rd64_tr16(uint32_t addr) {
  u32x2 v;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF) : "memory");
  return v;
}
template <int OFF>
__device__ __forceinline__ void lds_wr128(uint32_t addr, u32x4 v) {
  asm volatile("ds_write_b128 %0, %1 offset:%2" : : "v"(addr), "v"(v), "n"(OFF) : "memory");
}
__device__ __forceinline__ void lds_wr32(uint32_t addr, uint32_t v) {
  asm volatile("ds_write_b32 %0, %1" : : "v"(addr), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_wait() { asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory"); }
// values read by lds_rd* may be used only after lds_wait() and tie() of the variable
__device__ __forceinline__ void tie(u32x4& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void tie(uint32_t& v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void tie(u32x2& v) { asm volatile("" : "+v"(v)); }
template <class T, int N>
__device__ __forceinline__ void tie(T (&v)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) tie(v[i]);
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)(size_t)(const lds_char*)p;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x) {
  return __builtin_amdgcn_update_dpp(0.f, x, CTRL, 0xf, 0xf, false);
}
// rows listed in ROW_MASK receive the DPP source, the others keep x
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_rows(float x) {
  return __builtin_amdgcn_update_dpp(x, x, CTRL, ROW_MASK, 0xf, false);
}

// sum over aligned groups of LPR consecutive lanes; every lane of the group receives the result
template <int LPR>
__device__ __forceinline__ float group_sum(float x) {
  if constexpr (LPR >= 2) x += dpp_f<0xB1>(x);    // quad_perm [1,0,3,2]
  if constexpr (LPR >= 4) x += dpp_f<0x4E>(x);    // quad_perm [2,3,0,1]
  if constexpr (LPR >= 8) x += dpp_f<0x141>(x);   // row_half_mirror
  if constexpr (LPR >= 16) x += dpp_f<0x140>(x);  // row_mirror
  return x;
}
// e^d for d <= 0, the rounding of d * log2(e) put back in: exp2 of a product of ten is off by some 2e-7 without.
// (d = -inf: the remainder is no number and counts as -1, of nothing; no number stays none.)
__device__ __forceinline__ float exp_le0(float d) {
  const float e = d * LOG2E, r = __builtin_amdgcn_fmed3f(fmaf(d, LOG2E, -e), -1.0f, 1.0f), p = __builtin_amdgcn_exp2f(e);
  return fmaf(p, r * LN2, p);
}
__device__ __forceinline__ float rdlane(float x, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}

// whole-wave reductions: 16-lane rows by DPP, rows 0/1 and 2/3 by row_bcast15, halves by row_bcast31; lane 63 has
// the result, which is returned in a scalar register
// Whole-wave maxima of G values at once: 16-lane rows by DPP (quad swaps, half mirror, mirror), then row_bcast15
// (lane 15 of a row into the next row) and row_bcast31 (lane 31 into the upper half); afterwards LANE 63 ALONE holds
// the maximum of each value (the other lanes are not kept consistent by the last two steps).  The DPP form of v_max
// is written out because the compiler would put a quieting v_max and a separate DPP move around every step.  A DPP
// operand may not be read in the two instructions after the one that wrote it: the steps go value by value, so with
// three or more values the other values' instructions fill that gap, otherwise an s_nop does.  The values may come
// straight out of dot instructions, whose results an ordinary VALU instruction may not read for three instructions
// (the compiler pads its own code for this, not inline asm): hence the longer s_nop before the first step.  Source
// and destination are separate operands, so the register allocator has no reason to slip a copy in front of a step.
template <int G>
__device__ __forceinline__ void wave_max_all(float (&x)[G]) {
#define TKV_MAX_STEP(CTRL)                                                                             \
  _Pragma("unroll") for (int h = 0; h < G; ++h) {                                                      \
    float r;                                                                                           \
    if (G < 3 || h == 0) asm volatile("s_nop 1");                                                      \
    asm volatile("v_max_f32_dpp %0, %1, %1 " CTRL : "=v"(r) : "v"(x[h]));                              \
    x[h] = r;                                                                                          \
  }
  // every value is in its register before the first step, and its writer is far enough behind
  _Pragma("unroll") for (int h = 0; h < G; ++h) asm volatile("" : : "v"(x[h]));
  asm volatile("s_nop 3");
  TKV_MAX_STEP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
  TKV_MAX_STEP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
  TKV_MAX_STEP("row_half_mirror row_mask:0xf bank_mask:0xf")
  TKV_MAX_STEP("row_mirror row_mask:0xf bank_mask:0xf")
  TKV_MAX_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf")
  TKV_MAX_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf")
#undef TKV_MAX_STEP
}
// Sums of G values over aligned groups of 8 lanes, every lane of a group receiving the result; same scheme (and the
// same reason for writing the DPP form out) as wave_max_all.
template <int G>
__device__ __forceinline__ void group_sum8_all(float (&x)[G]) {
#define TKV_ADD_STEP(CTRL)                                                                             \
  _Pragma("unroll") for (int h = 0; h < G; ++h) {                                                      \
    float r;                                                                                           \
    if (G < 3 || h == 0) asm volatile("s_nop 1");                                                      \
    asm volatile("v_add_f32_dpp %0, %1, %1 " CTRL : "=v"(r) : "v"(x[h]));                              \
    x[h] = r;                                                                                          \
  }
  _Pragma("unroll") for (int h = 0; h < G; ++h) asm volatile("" : : "v"(x[h]));
  asm volatile("s_nop 3");
  TKV_ADD_STEP("quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf")
  TKV_ADD_STEP("quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf")
  TKV_ADD_STEP("row_half_mirror row_mask:0xf bank_mask:0xf")
#undef TKV_ADD_STEP
}
__device__ __forceinline__ float wave_sum(float x) {
  x = group_sum<16>(x);
  const float a = rdlane(x, 0) + rdlane(x, 16), b = rdlane(x, 32) + rdlane(x, 48);
  return a + b;
}

// Sums over the row groups of a wave: lane gv * LPRV + rv holds a partial of elements rv * EV + e (e < EV) for every group
// gv; afterwards the 64 lanes hold each total once, EV * LPRV / 64 per lane, element `elem` of the returned pairs.  Two
// values go through one swap of the wave's halves (then of its 16-lane rows, then of 8-lane half rows) and one addition:
// a fraction of what a shuffle per value costs (1.4 us for 56 values per lane, 0.2 us this way).
template <int EV, int LPRV>
struct RowSum { static constexpr int N = EV * LPRV / 64; };
__device__ __forceinline__ float add_swap32(float a, float b) {      // lanes 0..31: a's halves added; 32..63: b's
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
__device__ __forceinline__ float add_swap16(float a, float b) {      // even rows: a's row pair added; odd rows: b's
  const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
}
template <int EV, int LPRV>
__device__ __forceinline__ void row_sum(const float (&o)[EV], int lane, float (&t)[RowSum<EV, LPRV>::N]) {
  static_assert(LPRV == 8 || LPRV == 16 || LPRV == 32, "rows of 8, 16 or 32 lanes");
  float h[EV / 2];
#pragma unroll
  for (int k = 0; k < EV / 2; ++k) h[k] = add_swap32(o[2 * k], o[2 * k + 1]);
  if constexpr (LPRV == 32) {
#pragma unroll
    for (int k = 0; k < EV / 2; ++k) t[k] = h[k];
  } else {
    float q[EV / 4];
#pragma unroll
    for (int k = 0; k < EV / 4; ++k) q[k] = add_swap16(h[2 * k], h[2 * k + 1]);
    if constexpr (LPRV == 16) {
#pragma unroll
      for (int k = 0; k < EV / 4; ++k) t[k] = q[k];
    } else {
#pragma unroll
      for (int k = 0; k < EV / 8; ++k) {
        const float a = q[2 * k] + dpp_f<0x128>(q[2 * k]), b = q[2 * k + 1] + dpp_f<0x128>(q[2 * k + 1]);   // row_ror:8
        t[k] = (lane & 8) ? b : a;
      }
    }
  }
}
// element (within the row's D) of t[k] of this lane
template <int EV, int LPRV>
__device__ __forceinline__ int row_sum_elem(int lane, int k) {
  const int rv = lane % LPRV, hi = lane >> 5, odd = (lane >> 4) & 1, up = (lane >> 3) & 1;
  if constexpr (LPRV == 32) return rv * EV + 2 * k + hi;
  else if constexpr (LPRV == 16) return rv * EV + 4 * k + 2 * odd + hi;
  else return rv * EV + 8 * k + 4 * up + 2 * odd + hi;
}

__device__ __forceinline__ float bf_lo(uint32_t u) { return __builtin_bit_cast(float, u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __builtin_bit_cast(float, u & 0xffff0000u); }
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
// two code values (exact in binary16) packed as a binary16 pair
__device__ __forceinline__ uint32_t pack_f16_pair(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}
__device__ __forceinline__ float f16_lo(uint32_t u) { return (float)__builtin_bit_cast(f16x2, u).x; }
__device__ __forceinline__ float f16_hi(uint32_t u) { return (float)__builtin_bit_cast(f16x2, u).y; }
// two code values (exact in bf16: at most 8 significant bits) packed as a bf16 pair
__device__ __forceinline__ uint32_t pack_bf16_pair(float lo, float hi) {
  return (__builtin_bit_cast(uint32_t, hi) & 0xffff0000u) | (__builtin_bit_cast(uint32_t, lo) >> 16);
}
__device__ __forceinline__ float half_of(uint32_t w, int hi) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(hi ? (w >> 16) : (w & 0xffffu)));
}

// Logits of one call: [sequence entry][query head][xs_stride], by list index; scaled, but of one token on the matrix cores
// (split_on_matrix), whose readers scale them
__device__ __forceinline__ size_t xs_at(const AttnArgs& a, int seq, int hq, int col) {
  return ((size_t)seq * a.Hq + hq) * a.xs_stride + col;
}

template <int G>
struct GPad { static constexpr int v = (G <= 4) ? 4 : 8; };

// ---- geometry ------------------------------------------------------------------------------------------------
// A row is fetched in "units" of 16 bytes (4 bytes where a lane's share of a row is shorter than 16), one unit per
// lane and direct-to-LDS instruction; the lane that fetched a unit is the lane that reads it back.
//   K side: 8 lanes per row; lane r8 owns units j*8 + r8, j < KU          (K batch i = rows NB*g8 + i, g8 = lane/8)
//   V side: LPRV lanes per row; lane rv owns units rv*VU + u, u < VU      (V step it = rows NITV*gv + it, gv = lane/LPRV)
// TR rows per tile (64, or fewer where a wave has less LDS); with TR < 64 the lanes r8 >= TR / 8 carry no entry of their own.
template <int D, Mode M, int TR = 64>
struct Geo {
  static constexpr bool IS_Q = (M == Q_INT8 || M == Q_INT4);
  static constexpr int RB = (M == F_BF16 || M == F_F16) ? 2 * D : (M == F_F32) ? 4 * D : (M == Q_INT8) ? D : D / 2;   // bytes per row
  static constexpr int KLB = RB / 8;                        // bytes of a K row per lane
  static constexpr int KS = (KLB % 16 == 0) ? 16 : 4;       // bytes per unit
  static constexpr int KU = KLB / KS;                       // units per lane and row
  static constexpr int EUK = KS * D / RB;                   // elements per unit
  static constexpr int EV = (M == F_F32) ? 4 : 8;           // elements of a V row per lane
  static constexpr int LPRV = D / EV;                       // lanes per V row
  static constexpr int NB = TR / 8;                         // K batches per tile
  static constexpr int NITV = TR * LPRV / 64;               // V steps per tile
  static constexpr int VLB = RB / LPRV;                     // bytes of a V row per lane
  static constexpr int VS = (VLB % 16 == 0) ? 16 : 4;
  static constexpr int VU = VLB / VS;
  static constexpr int EUV = EV / VU;                       // elements per V unit
  static constexpr int SCD = (M == Q_INT8) ? 1 : (M == Q_INT4) ? D / 64 : 0;   // dwords of scales per row
  // direct-to-LDS operations of one tile period: slot list, K scales, N_K K pieces, V scales, N_V V pieces
  static constexpr int N_K = NB * KU, N_V = NITV * VU;
  static_assert(KLB % KS == 0 && VLB % VS == 0 && NITV % 4 == 0 && NB % 4 == 0 && (!IS_Q || D % 64 == 0), "unsupported head_dim");
};

template <int S>
struct UnitT { using type = uint32_t; };
template <>
struct UnitT<16> { using type = u32x4; };

// element c of a vector, by value (a bit cast applied directly to a vector element reads element 0)
__device__ __forceinline__ uint32_t elem(const u32x4& v, int c) { return v[c]; }
__device__ __forceinline__ float elem_f(const u32x4& v, int c) { const uint32_t w = v[c]; return __builtin_bit_cast(float, w); }

template <int S>
__device__ __forceinline__ uint32_t unit_word(const typename UnitT<S>::type& u, int c) {
  if constexpr (S == 16) return u[c]; else return u;
}

// Codes of one unit, sign-extended.  (Read as unsigned code + offset, with the offset taken out of a wave's finished sums,
// they cost a wave that walks many rows its last bits: the offsets' share of a sum grows with the rows, the sum itself with
// their square root.  One workgroup per pair, 6000 tokens of which 15 % int4: outputs 9.7e-7 off 64 bits, 3.5e-7 so.)
template <Mode M, int S, int E>
__device__ __forceinline__ void unpack_unit(const typename UnitT<S>::type& u, float (&f)[E]) {
  if constexpr (M == Q_INT8) {
#pragma unroll
    for (int i = 0; i < S / 4; ++i) {
      const uint32_t w = unit_word<S>(u, i);
#pragma unroll
      for (int n = 0; n < 4; ++n) f[i * 4 + n] = (float)(int8_t)(w >> (8 * n));
    }
  } else {
#pragma unroll
    for (int i = 0; i < S / 4; ++i) {
      const uint32_t w = unit_word<S>(u, i);
#pragma unroll
      for (int n = 0; n < 8; ++n) f[i * 8 + n] = (float)((int32_t)(w << (28 - 4 * n)) >> 28);
    }
  }
}

// The lane's units of the G query vectors.  bf16 queries stay packed (fed to the bf16 dot instruction); binary32
// queries are kept as floats.
template <int D, int G, Mode M, int KT>
struct QRegs {
  using GE = Geo<D, M>;
  static constexpr bool QBF = KT != KT_F32;   // 16-bit queries stay packed in pairs
  uint32_t qp[QBF ? G : 1][GE::KU][GE::EUK / 2];
  float qf[QBF ? 1 : G][GE::KU][GE::EUK];
};

template <int D, Mode M>
struct KBatch { typename UnitT<Geo<D, M>::KS>::type u[Geo<D, M>::KU]; };
template <int D, int G, Mode M>
struct VStep {
  typename UnitT<Geo<D, M>::VS>::type u[Geo<D, M>::VU];
  u32x4 p[GPad<G>::v / 4];
};

// G logits of one K row, reduced over the row's 8 lanes (every lane of the group gets them).
// sc: INT8 the row's scale; INT4 the scale of the 32-code group of each of the lane's units.
template <int D, int G, Mode M, int KT>
__device__ __forceinline__ void row_logits(const KBatch<D, M>& kr, const QRegs<D, G, M, KT>& q,
                                           const float (&sc)[Geo<D, M>::KU], float (&x)[G]) {
  using GE = Geo<D, M>;
  constexpr int KU = GE::KU, KS = GE::KS, EUK = GE::EUK;
  constexpr bool QBF = KT != KT_F32, H = KT == KT_F16;
  if constexpr (M == F_F16) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j < KU; ++j)
#pragma unroll
        for (int c = 0; c < EUK / 2; ++c)
          acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, unit_word<KS>(kr.u[j], c)),
                                       __builtin_bit_cast(f16x2, q.qp[h][j][c]), acc, false);
      x[h] = acc;
    }
    group_sum8_all<G>(x);
  } else if constexpr (M == F_BF16) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j < KU; ++j)
#pragma unroll
        for (int c = 0; c < EUK / 2; ++c)
          acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, unit_word<KS>(kr.u[j], c)),
                                                __builtin_bit_cast(bf16x2, q.qp[h][j][c]), acc, false);
      x[h] = acc;
    }
    group_sum8_all<G>(x);
  } else if constexpr (M == F_F32) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      float acc = 0.f;
#pragma unroll
      for (int j = 0; j < KU; ++j)
#pragma unroll
        for (int c = 0; c < EUK; ++c) acc = fmaf(__builtin_bit_cast(float, unit_word<KS>(kr.u[j], c)), q.qf[h][j][c], acc);
      x[h] = acc;
    }
    group_sum8_all<G>(x);
  } else {
    float tot[G];
#pragma unroll
    for (int h = 0; h < G; ++h) tot[h] = 0.f;
#pragma unroll
    for (int j = 0; j < KU; ++j) {
      float kf[EUK];
      unpack_unit<M, KS, EUK>(kr.u[j], kf);
      uint32_t kp[EUK / 2];
      if constexpr (QBF) {
#pragma unroll
        for (int c = 0; c < EUK / 2; ++c) kp[c] = H ? pack_f16_pair(kf[2 * c], kf[2 * c + 1]) : pack_bf16_pair(kf[2 * c], kf[2 * c + 1]);
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float acc = 0.f;
        if constexpr (QBF) {
#pragma unroll
          for (int c = 0; c < EUK / 2; ++c) {
            if constexpr (H) acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, kp[c]), __builtin_bit_cast(f16x2, q.qp[h][j][c]), acc, false);
            else acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, kp[c]), __builtin_bit_cast(bf16x2, q.qp[h][j][c]), acc, false);
          }
        } else {
#pragma unroll
          for (int c = 0; c < EUK; ++c) acc = fmaf(q.qf[h][j][c], kf[c], acc);
        }
        if constexpr (M == Q_INT4) tot[h] = fmaf(acc, sc[j], tot[h]);   // per-group scale: before the cross-lane sum
        else tot[h] += acc;
      }
    }
    group_sum8_all<G>(tot);
#pragma unroll
    for (int h = 0; h < G; ++h) {
      x[h] = tot[h];
      if constexpr (M == Q_INT8) x[h] *= sc[0];                         // per-row scale
    }
  }
}

// o[h][e] += p[h] * v[e] for the lane's EV elements of one V row (Q modes: p scaled)
template <int D, int G, Mode M>
__device__ __forceinline__ void row_accumulate(const VStep<D, G, M>& vr, float sc, float (&o)[G][Geo<D, M>::EV]) {
  using GE = Geo<D, M>;
  constexpr int EV = GE::EV, VU = GE::VU, VS = GE::VS, EUV = GE::EUV;
  float p[GPad<G>::v];
#pragma unroll
  for (int c = 0; c < GPad<G>::v; ++c) p[c] = elem_f(vr.p[c / 4], c % 4);
  float vf[EV];
  if constexpr (M == F_BF16) {
#pragma unroll
    for (int c = 0; c < 4; ++c) { const uint32_t wv = elem(vr.u[0], c); vf[2 * c] = bf_lo(wv); vf[2 * c + 1] = bf_hi(wv); }
  } else if constexpr (M == F_F16) {
#pragma unroll
    for (int c = 0; c < 4; ++c) { const uint32_t wv = elem(vr.u[0], c); vf[2 * c] = f16_lo(wv); vf[2 * c + 1] = f16_hi(wv); }
  } else if constexpr (M == F_F32) {
#pragma unroll
    for (int c = 0; c < 4; ++c) vf[c] = elem_f(vr.u[0], c);
  } else {
#pragma unroll
    for (int u = 0; u < VU; ++u) {
      float t[EUV];
      unpack_unit<M, VS, EUV>(vr.u[u], t);
#pragma unroll
      for (int e = 0; e < EUV; ++e) vf[u * EUV + e] = t[e];
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float ph = p[h];
    if constexpr (GE::IS_Q) ph *= sc;
#pragma unroll
    for (int e = 0; e < EV; ++e) o[h][e] = fmaf(ph, vf[e], o[h][e]);
  }
}

// LDS regions of one wave (pointers for the direct loads, byte addresses for the reads)
struct WaveLds {
  char* t; char* sk; char* sv; char* lt;   // tile buffer (K rows, then V rows, in turn), K scales, V scales, slot lists (2 x 64 ints)
  char* p;                                 // probabilities of the current tile (before the first tile: the query block)
  uint32_t ta, ska, sva, lta, pa;          // the same as LDS addresses
  uint32_t lga; int lcap, lim;             // k_attn_step: logits [G][lcap] in LDS; the columns from lim (whole tiles: lcap, or
  float* sp; int sp_stride;                // none for a part of a pair) on go to memory, column c of head h to sp[h * sp_stride + c]
};

struct __attribute__((packed, aligned(2))) PackedU32x4 { u32x4 v; };   // 16 bytes at any 16-bit element

template <int SZ>
__device__ __forceinline__ void dma(const __amdgpu_buffer_rsrc_t& rs, char* lds, uint32_t voff, int aux) {
  static_assert(SZ == 16 || SZ == 4, "unit sizes");
  if constexpr (SZ == 16) {
    if (aux) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)lds, 16, voff, 0, 0, 2);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)lds, 16, voff, 0, 0, 0);
  } else {
    if (aux) __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)lds, 4, voff, 0, 0, 2);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)lds, 4, voff, 0, 0, 0);
  }
}

// ---- one wave: the tiles tile0, tile0 + tstride, ... of one list ------------------------------------------------
// One tile buffer per wave holds the K rows of a tile, then its V rows, then the next tile's K rows: a K batch that
// has been read is refilled with the V pieces that fall on the same bytes, a V step with K pieces of the next tile.
// Issue order of one tile period (the vmcnt arguments below are counts of younger operations in this order):
//   slot list of tile t+2 | K scales of t+1 | per K batch of t: the V pieces of t on its bytes |
//   V scales of t+1 | per V step of t: the K pieces of t+1 on its bytes
// Accumulates into o, m_run, l_lane (per-lane partial sums of the softmax denominator, relative to m_run); leaves the
// scaled logits in xs (WHOLE, k_attn_step: unscaled ones in the LDS, which has room for all).
template <int D, int G, Mode M, int KT, int TR, bool WHOLE = false>
__device__ __forceinline__ void attn_wave(const AttnArgs& a, const WaveLds& w, int b, int jq, int kvh, int lane,
                                          int tile0, int tstride, int n_list, const int* loc_list, int col0,
                                          float (&o)[G][Geo<D, M>::EV], float (&m_run)[G], float (&l_lane)[G]) {
  using GE = Geo<D, M, TR>;
  constexpr int NB = GE::NB;
  constexpr int EV = GE::EV, LPRV = GE::LPRV, NITV = GE::NITV, KU = GE::KU, KS = GE::KS, VU = GE::VU, VS = GE::VS;
  constexpr int EUK = GE::EUK, SCD = GE::SCD, RB = GE::RB, N_K = GE::N_K, N_V = GE::N_V;
  constexpr int GP = GPad<G>::v;
  constexpr bool QBF = KT != KT_F32;
  constexpr int KIB = 64 * KS, VIB = 64 * VS;        // bytes of the tile buffer one K / V piece covers
  constexpr int KBB = KU * KIB, VSB = VU * VIB;      // ... one K batch / one V step
  static_assert(KBB % VIB == 0 && NB * KBB == NITV * VSB, "K batches and V steps tile the same buffer");
  constexpr int VPB = KBB / VIB;                     // V pieces issued after each K batch
  const int g8 = lane >> 3, r8 = lane & 7;           // K side: row group and unit column
  const int gv = lane / LPRV, rv = lane % LPRV;      // V side
  const int entry = NB * g8 + r8;                    // the tile's entry whose logits this lane keeps
  const bool keeps = NB == 8 || r8 < NB;

  __amdgpu_buffer_rsrc_t rk, rvv, rsk, rsv;
  if constexpr (!GE::IS_Q) {
    const size_t off = (size_t)(b * a.Hkv + kvh) * a.capF * RB;
    rk = make_rsrc(a.fpK + off, (uint32_t)a.capF * RB); rvv = make_rsrc(a.fpV + off, (uint32_t)a.capF * RB);
    rsk = rk; rsv = rvv;
  } else {
    const size_t rows = (size_t)(b * a.Hkv + kvh) * a.cap2;
    rk = make_rsrc(a.c2K + rows * a.cb, (uint32_t)a.cap2 * a.cb); rvv = make_rsrc(a.c2V + rows * a.cb, (uint32_t)a.cap2 * a.cb);
    rsk = make_rsrc(a.s2K + rows * a.sb, (uint32_t)a.cap2 * a.sb); rsv = make_rsrc(a.s2V + rows * a.sb, (uint32_t)a.cap2 * a.sb);
  }
  const __amdgpu_buffer_rsrc_t rl = make_rsrc(loc_list, (uint32_t)a.Nmax * 4u);

  if (tile0 * TR >= n_list) return;

  // a tile's slot list and scales: one dword per lane and entry (lanes past the tile's rows stay out of it)
  auto issue_loc = [&](int par, int tile) {
    if (TR == 64 || lane < TR) dma<4>(rl, w.lt + par * (TR * 4), (uint32_t)(tile * TR + lane) * 4u, 0);
  };
  // The first tile's slot list is asked for before anything else: the compute unit serves its waves' requests in
  // the order they were made, and a list request that came behind another wave's rows would wait for all of them.
  issue_loc(0, tile0);

  // The lane's units of the G query vectors.  16-bit queries (G * D * 2 bytes, contiguous) come in through the
  // probability region of the LDS, as NQD direct loads of 1 KB whose count the waits below can name; binary32
  // queries are fetched by ordinary loads (the wait for the list then waits for them as well).
  QRegs<D, G, M, KT> q;
  constexpr bool QLDS = QBF && (G * D * 2 + 1023) / 1024 * 1024 <= TR * GP * 4;
  constexpr int NQD = QLDS ? (G * D * 2 + 1023) / 1024 : 0;
  if constexpr (QBF && !QLDS) {
    // no room for the block in the probability region: ordinary loads, which the wait for the list then waits for as well
    const char* qb = (const char*)a.q + ((size_t)b * a.q_bs + (size_t)jq * a.Hq + kvh * G) * D * 2;
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        const uint32_t* src = (const uint32_t*)(qb + ((size_t)h * D + (size_t)(j * 8 + r8) * EUK) * 2);
#pragma unroll
        for (int c = 0; c < EUK / 2; ++c) q.qp[h][j][c] = src[c];
      }
  } else if constexpr (QLDS) {
    const char* qb = (const char*)a.q + ((size_t)b * a.q_bs + (size_t)jq * a.Hq + kvh * G) * D * 2;
    if (((uintptr_t)a.q & 15) == 0) {
      const __amdgpu_buffer_rsrc_t rq = make_rsrc(qb, (uint32_t)(G * D * 2));   // lanes past the block fetch zeros
#pragma unroll
      for (int i = 0; i < NQD; ++i) dma<16>(rq, w.p + i * 1024, (uint32_t)(i * 1024 + lane * 16), 0);
    } else {                                             // (queries that begin between 16-byte boundaries: plain loads; none is left to wait for)
#pragma unroll
      for (int i = 0; i < NQD; ++i)
        if (i * 1024 + lane * 16 < G * D * 2) lds_wr128<0>(w.pa + (uint32_t)(i * 1024 + lane * 16), ((const PackedU32x4*)(qb + i * 1024 + lane * 16))->v);
    }
  } else {
    const char* qb = (const char*)a.q + ((size_t)b * a.q_bs + (size_t)jq * a.Hq + kvh * G) * D * 4;
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int j = 0; j < KU; ++j) {
        const char* src = qb + ((size_t)h * D + (size_t)(j * 8 + r8) * EUK) * 4;
#pragma unroll
        for (int c = 0; c < EUK; ++c) q.qf[h][j][c] = ((const float*)src)[c];
      }
  }

  // per-lane byte offsets of its units within a row, and its LDS read addresses
  const uint32_t kcol = (uint32_t)r8 * KS, vcol = (uint32_t)rv * (VU * VS);
  const uint32_t k_rd = w.ta + (uint32_t)lane * KS, v_rd = w.ta + (uint32_t)lane * VS;
  const uint32_t p_wr = w.pa + (uint32_t)entry * (GP * 4), p_rd = w.pa + (uint32_t)(gv * NITV) * (GP * 4);

  // slots of the rows this lane fetches: lk / lrow belong to the tile whose K rows are fetched next, lv to the
  // tile whose V rows are fetched next
  int lk[NB], lv[NITV], lrow;
  // reads the K-side slots (rows NB*g8 + i) and the lane's own row's slot of the list in LDS half `par`
  auto read_locs_k = [&](int par, int nvalid) {
    const uint32_t base = w.lta + (uint32_t)par * (TR * 4u);
    if (nvalid < TR) {                                   // wave-uniform: a list's last tile
      if (lane >= nvalid && lane < TR) lds_wr32(base + (uint32_t)lane * 4u, 0xffffffffu);   // no row: fetches land as zeros
    }
    u32x4 t[NB / 4];
    static_for<NB / 4>([&](auto cc) { constexpr int c = decltype(cc)::value; t[c] = lds_rd128<c * 16>(base + (uint32_t)g8 * (NB * 4u)); });
    uint32_t me = lds_rd32<0>(base + (uint32_t)(lane & (TR - 1)) * 4u);
    lds_wait(); tie(t); tie(me);
#pragma unroll
    for (int c = 0; c < NB / 4; ++c) { lk[4 * c] = t[c].x; lk[4 * c + 1] = t[c].y; lk[4 * c + 2] = t[c].z; lk[4 * c + 3] = t[c].w; }
    lrow = (int)me;
  };
  auto read_locs_v = [&](int par) {
    const uint32_t base = w.lta + (uint32_t)par * (TR * 4u) + (uint32_t)(gv * NITV) * 4u;
    u32x4 t[NITV / 4];
    static_for<NITV / 4>([&](auto cc) { constexpr int c = decltype(cc)::value; t[c] = lds_rd128<c * 16>(base); });
    lds_wait(); tie(t);
#pragma unroll
    for (int c = 0; c < NITV / 4; ++c) { lv[4 * c] = t[c].x; lv[4 * c + 1] = t[c].y; lv[4 * c + 2] = t[c].z; lv[4 * c + 3] = t[c].w; }
  };
  auto issue_kscale = [&]() {
    if (TR == 64 || lane < TR) {
#pragma unroll
      for (int j = 0; j < SCD; ++j) dma<4>(rsk, w.sk + j * (TR * 4), (uint32_t)lrow * (uint32_t)a.sb + j * 4u, 0);
    }
  };
  auto issue_vscale = [&]() {
    if (TR == 64 || lane < TR) {
#pragma unroll
      for (int j = 0; j < SCD; ++j) dma<4>(rsv, w.sv + j * (TR * 4), (uint32_t)lrow * (uint32_t)a.sb + j * 4u, 0);
    }
  };
  auto issue_k_piece = [&](int s) {                      // K piece s = (batch s / KU, unit s % KU)
    const int i = s / KU, j = s % KU;
    dma<KS>(rk, w.t + s * KIB, (uint32_t)lk[i] * (uint32_t)RB + (uint32_t)j * (8 * KS) + kcol, 1);
  };
  auto issue_v_piece = [&](int v) {                      // V piece v = (step v / VU, unit v % VU)
    const int it = v / VU, u = v % VU;
    dma<VS>(rvv, w.t + v * VIB, (uint32_t)lv[it] * (uint32_t)RB + vcol + (uint32_t)u * VS, 1);
  };

  // ---- prologue: the first tile's slot list has been asked for; then its scales and K rows in the order of a tile
  // period, and the query block out of the LDS into registers
  wait_vm<NQD>();                                        // the list is in (binary32 queries: and the queries)
  read_locs_k(0, n_list - tile0 * TR);
  issue_loc(1, tile0 + tstride);
  issue_kscale();
  issue_vscale();
#pragma unroll
  for (int s = 0; s < N_K; ++s) issue_k_piece(s);
  if constexpr (QLDS) {
    wait_vm<1 + 2 * SCD + N_K>();                        // everything older than the second list: the query block
    // a unit of a query is EUK 16-bit elements: 8 bytes (one ds_read_b64) or QB pieces of 16
    constexpr int QW = EUK / 2, QB = QW / 4;
    static_assert(QW == 2 || QW % 4 == 0, "query units are 8 bytes or whole 16-byte pieces");
    const uint32_t q_rd = w.pa + (uint32_t)r8 * (EUK * 2);
    if constexpr (QW == 2) {
      u32x2 t[G][KU];
      static_for<G>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        static_for<KU>([&](auto jc) { constexpr int j = decltype(jc)::value; t[h][j] = lds_rd64<h * D * 2 + j * 8 * EUK * 2>(q_rd); });
      });
      lds_wait();
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int j = 0; j < KU; ++j) { tie(t[h][j]); q.qp[h][j][0] = t[h][j].x; q.qp[h][j][1] = t[h][j].y; }
    } else {
      u32x4 t[G][KU][QB > 0 ? QB : 1];
      static_for<G>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        static_for<KU>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          static_for<QB>([&](auto cc) { constexpr int c = decltype(cc)::value; t[h][j][c] = lds_rd128<h * D * 2 + j * 8 * EUK * 2 + c * 16>(q_rd); });
        });
      });
      lds_wait();
#pragma unroll
      for (int h = 0; h < G; ++h)
#pragma unroll
        for (int j = 0; j < KU; ++j)
#pragma unroll
          for (int c = 0; c < QB; ++c) {
            tie(t[h][j][c]);
#pragma unroll
            for (int e = 0; e < 4; ++e) q.qp[h][j][c * 4 + e] = elem(t[h][j][c], e);
          }
    }
  }

  int par = 1;                                           // LDS half that holds the next tile's slot list
  auto tile_body = [&](int tile, auto more_c) {
    constexpr bool MORE = decltype(more_c)::value;
    constexpr int X = MORE ? 1 : 0;                      // operations of the parts a last tile does not issue
    const bool valid = keeps && tile * TR + entry < n_list;
    // The two waves of a SIMD are issued oldest first, which lets the first wave of a pair run a whole tile ahead and
    // leaves the second one to finish on its own; the wave with more phases still to do goes first instead.
    __builtin_amdgcn_s_setprio(MORE ? 3 : 1);
    // -- V-side slots of this tile; K-side slots of the next one; fetch the list after that
    read_locs_v(par ^ 1);
    if constexpr (MORE) {
      wait_vm<2 * SCD + N_K>();
      read_locs_k(par, n_list - (tile + tstride) * TR);
      issue_loc(par ^ 1, tile + 2 * tstride);
    }
    // -- K scales of this tile
    float ksc[NB][KU];
    if constexpr (GE::IS_Q) {
      wait_vm<SCD + N_K + X>();
      u32x4 t[SCD][NB / 4];
      static_for<SCD>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        static_for<NB / 4>([&](auto cc) { constexpr int c = decltype(cc)::value; t[j][c] = lds_rd128<j * (TR * 4) + c * 16>(w.ska + (uint32_t)g8 * (NB * 4u)); });
      });
      lds_wait();
#pragma unroll
      for (int j = 0; j < SCD; ++j) tie(t[j]);
      if constexpr (MORE) issue_kscale();
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < KU; ++j) {
          if constexpr (M == Q_INT8) ksc[i][j] = elem_f(t[0][i / 4], i % 4);
          else ksc[i][j] = half_of(elem(t[j][i / 4], i % 4), (r8 >> 2) & 1);   // unit j*8 + r8 lies in group 2*j + r8/4
        }
    }
    // -- K rows: read batch i+1 while batch i is computed; a batch that has been read is refilled with V pieces
    float xt[G];
#pragma unroll
    for (int h = 0; h < G; ++h) xt[h] = 0.f;
    KBatch<D, M> kb[2];
    auto read_k = [&](auto ic, KBatch<D, M>& dst) {
      constexpr int i = decltype(ic)::value;
      // younger than this batch's pieces: the later K pieces, the list and K-scale fetches of this period, the V pieces so far
      wait_vm<N_K - 1 - ((i + 1) * KU - 1) + X * (1 + SCD) + i * VPB>();
      static_for<KU>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        if constexpr (KS == 16) dst.u[j] = lds_rd128<(i * KU + j) * KIB>(k_rd);
        else dst.u[j] = lds_rd32<(i * KU + j) * KIB>(k_rd);
      });
    };
    read_k(std::integral_constant<int, 0>{}, kb[0]);
    static_for<NB>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      lds_wait(); tie(kb[i & 1].u);
#pragma unroll
      for (int v = i * VPB; v < (i + 1) * VPB; ++v) issue_v_piece(v);
      if constexpr (i + 1 < NB) read_k(std::integral_constant<int, (i + 1 < NB ? i + 1 : NB - 1)>{}, kb[(i + 1) & 1]);
      float x[G];
      row_logits<D, G, M, KT>(kb[i & 1], q, ksc[i], x);
#pragma unroll
      for (int h = 0; h < G; ++h) xt[h] = (r8 == i) ? x[h] : xt[h];   // lane 8*g8 + i keeps entry NB*g8 + i
    });
    // -- online softmax, one entry per lane; the denominator is summed per lane and reduced once at the end
    float corr[G];
    {
      const int col = col0 + tile * TR + entry;
      float pv[GP];
#pragma unroll
      for (int h = 0; h < GP; ++h) pv[h] = 0.f;
      float x[G], xm[G];
#pragma unroll
      for (int h = 0; h < G; ++h) {
        x[h] = valid ? xt[h] * a.softmax_scale : -INFINITY;
        xm[h] = x[h];
      }
      if constexpr (WHOLE) {
        if (valid) {
#pragma unroll
          for (int h = 0; h < G; ++h) lds_wr32(w.lga + (uint32_t)(h * w.lcap + col) * 4u, __builtin_bit_cast(uint32_t, xt[h]));
        }
      } else if (valid) {
        const size_t xbase = xs_at(a, b * a.n_q + jq, kvh * G, col);
#pragma unroll
        for (int h = 0; h < G; ++h) a.xs[xbase + (size_t)h * a.xs_stride] = x[h];
      }
      wave_max_all<G>(xm);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        // m_run starts at -inf: corr = exp2(-inf) = 0 there, against zero accumulators.  Tiles whose logits are all -inf
        // leave it there: their weights are exp2(-inf) = 0 too.
        const float mn = fmaxf(m_run[h], rdlane(xm[h], 63)), ms = mn > -INFINITY ? mn : 0.f;
        corr[h] = __builtin_amdgcn_exp2f((m_run[h] - ms) * LOG2E);
        const float p = valid ? __builtin_amdgcn_exp2f((x[h] - ms) * LOG2E) : 0.f;
        l_lane[h] = fmaf(l_lane[h], corr[h], p);
        m_run[h] = mn;
        pv[h] = p;
      }
      if (keeps) static_for<GP / 4>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        u32x4 t;
        t.x = __builtin_bit_cast(uint32_t, pv[4 * c]); t.y = __builtin_bit_cast(uint32_t, pv[4 * c + 1]);
        t.z = __builtin_bit_cast(uint32_t, pv[4 * c + 2]); t.w = __builtin_bit_cast(uint32_t, pv[4 * c + 3]);
        lds_wr128<c * 16>(p_wr, t);
      });
    }
    {
      // the running maxima are wave-uniform; once they have settled no head needs rescaling (x * 1.0f is exact)
      bool moved = false;
#pragma unroll
      for (int h = 0; h < G; ++h) moved = moved || (corr[h] != 1.0f);
      if (moved) {
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
          for (int e = 0; e < EV; ++e) o[h][e] *= corr[h];
      }
    }
    // -- V scales of this tile
    __builtin_amdgcn_s_setprio(MORE ? 2 : 0);
    float vsc[NITV];
    if constexpr (GE::IS_Q) {
      wait_vm<N_K + X * (1 + SCD) + N_V>();
      const uint32_t base = w.sva + (uint32_t)(gv * NITV) * 4u + ((M == Q_INT4) ? (uint32_t)(rv >> 3) * (TR * 4u) : 0u);
      u32x4 t[NITV / 4];
      static_for<NITV / 4>([&](auto cc) { constexpr int c = decltype(cc)::value; t[c] = lds_rd128<c * 16>(base); });
      lds_wait(); tie(t);
      if constexpr (MORE) issue_vscale();
#pragma unroll
      for (int it = 0; it < NITV; ++it) {
        if constexpr (M == Q_INT8) vsc[it] = elem_f(t[it / 4], it % 4);
        else vsc[it] = half_of(elem(t[it / 4], it % 4), (rv >> 2) & 1);        // unit rv lies in group rv/4
      }
    }
    // -- V rows: a step that has been read is refilled with the next tile's K pieces that fall on its bytes
    VStep<D, G, M> vb[2];
    auto read_v = [&](auto ic, VStep<D, G, M>& dst) {
      constexpr int it = decltype(ic)::value;
      // younger than this step's pieces: the later V pieces, the V-scale fetches of this period, the K pieces so far
      wait_vm<N_V - 1 - ((it + 1) * VU - 1) + X * (SCD + (it * VSB) / KIB)>();
      static_for<VU>([&](auto uc) {
        constexpr int u = decltype(uc)::value;
        if constexpr (VS == 16) dst.u[u] = lds_rd128<(it * VU + u) * VIB>(v_rd);
        else dst.u[u] = lds_rd32<(it * VU + u) * VIB>(v_rd);
      });
      static_for<GP / 4>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        dst.p[c] = lds_rd128<it * GP * 4 + c * 16>(p_rd);
      });
    };
    read_v(std::integral_constant<int, 0>{}, vb[0]);
    static_for<NITV>([&](auto ic) {
      constexpr int it = decltype(ic)::value;
      lds_wait(); tie(vb[it & 1].u); tie(vb[it & 1].p);
      if constexpr (MORE) {
#pragma unroll
        for (int s = (it * VSB) / KIB; s < ((it + 1) * VSB) / KIB; ++s) issue_k_piece(s);
      }
      if constexpr (it + 1 < NITV) read_v(std::integral_constant<int, (it + 1 < NITV ? it + 1 : NITV - 1)>{}, vb[(it + 1) & 1]);
      row_accumulate<D, G, M>(vb[it & 1], GE::IS_Q ? vsc[it] : 0.f, o);
    });
    par ^= 1;
  };

  int tile = tile0;
  for (; (tile + tstride) * TR < n_list; tile += tstride) tile_body(tile, std::true_type{});
  tile_body(tile, std::false_type{});
}

// ---- one wave on the matrix cores: tiles of list F with 16-bit rows ------------------------------------------------
//   logits  : C[entry][column] = K[entry][:] . q[column][:], 16 entries per instruction, D/32 instructions deep.  Lane
//             (column = lane % 16, kb = lane / 16) ends up with the logits of entries 16*rb + 4*kb + 0..3 of its column,
//             which is exactly the layout of the left operand of the second product, so the probabilities never leave
//             the registers.
//   softmax : online per column; a quarter of a tile's entries per lane, the maximum completed over the column's 4 lanes.
//   output  : O[column][d] += P[column][entry] * V[entry][d], 32 entries per instruction; the right operand needs, per
//             lane, the same column of 4 + 4 rows: a transposing LDS read delivers it.  P is fed as two or three 16-bit
//             terms (PSplit).
// Rows still come in by direct-to-LDS loads of 1 KB (8 rows x 8 pieces of 16 bytes, 128 contiguous bytes per row).
// Within a row's 128 bytes the pieces are rotated by an amount that depends on the row, so that the 16 lanes of an
// operand read (16 different rows, same piece) fall on 16 different bank groups; the rotation is undone by the read
// addresses.  K rows of a tile, its V rows and the next tile's K rows pass through the one tile buffer as in attn_wave:
// the K rows of 16 entries are replaced by V pieces once read, half a tile of V rows by the next tile's K pieces.
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

template <int KT>
__device__ __forceinline__ f32x4 mfma_16x16x32(const u32x4& x, const u32x4& y, f32x4 c) {
  if constexpr (KT == KT_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x), __builtin_bit_cast(bf16x8, y), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, x), __builtin_bit_cast(f16x8, y), c, 0, 0, 0);
}
// the same, 16 deep: operands of 8 bytes a lane
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
template <int KT>
__device__ __forceinline__ f32x4 mfma_16x16x16(const u32x2& x, const u32x2& y, f32x4 c) {
  if constexpr (KT == KT_BF16)
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, x), __builtin_bit_cast(s16x4, y), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(f16x4, x), __builtin_bit_cast(f16x4, y), c, 0, 0, 0);
}
// maximum / sum over the four lanes n, n + 16, n + 32, n + 48, in all of them
__device__ __forceinline__ float quad_max(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  x = fmaxf(__builtin_bit_cast(float, (uint32_t)h[0]), __builtin_bit_cast(float, (uint32_t)h[1]));
  const uint32_t v = __builtin_bit_cast(uint32_t, x);
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}
__device__ __forceinline__ float quad_sum(float x) {
  x = add_swap32(x, x);
  return add_swap16(x, x);
}
// quotient of small non-negative integers (below 2^13): exact, a conversion and a product instead of a division
__device__ __forceinline__ int small_div(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }

// A binary32 weight as a sum of 16-bit terms, each the leading bits (by truncation) of what the terms before it left.
// bfloat16: three terms of 8 significant bits are the weight exactly.  binary16: two terms of 11 bits (22 of the 24);
// the weights are taken times 2^P_SHIFT there, so that small ones stay clear of binary16's narrow exponent range
// (the factor is taken out of the accumulators at the end).  One query token: three terms in either type, and binary16's
// weights relative to the tile's largest (attn_wave_mfma).
template <int KT>
struct PSplit {
  static constexpr int N = KT == KT_BF16 ? 3 : 2;
  static constexpr float P_SHIFT = KT == KT_BF16 ? 0.f : 14.f;
  static constexpr float SCALE_MAX = 3.75f;   // binary16: what a weight of 1 can be multiplied by and stay in range (65504) with the shift
};
// (p0, p1: left with what the terms do not hold)
template <int KT, int N>
__device__ __forceinline__ void split_pair(float& p0, float& p1, uint32_t (&t)[N]) {
  if constexpr (KT == KT_BF16) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const uint32_t u0 = __builtin_bit_cast(uint32_t, p0) & 0xffff0000u, u1 = __builtin_bit_cast(uint32_t, p1) & 0xffff0000u;
      t[i] = u1 | (u0 >> 16);
      p0 -= __builtin_bit_cast(float, u0);
      p1 -= __builtin_bit_cast(float, u1);
    }
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const f16x2 h = __builtin_bit_cast(f16x2, __builtin_amdgcn_cvt_pkrtz(p0, p1));
      t[i] = __builtin_bit_cast(uint32_t, h);
      p0 -= (float)h.x;
      p1 -= (float)h.y;
    }
  }
}

// Code values (one byte each, or two per byte) as 16-bit floating point, sign-extended: at most 7 significant bits, so the
// matrix cores multiply them exactly.  Two values per 32-bit word, low element first.
template <int KT>
__device__ __forceinline__ uint32_t pack16(float lo, float hi) {
  if constexpr (KT == KT_BF16) return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, hi), __builtin_bit_cast(uint32_t, lo), 0x07060302u);
  else return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}
__device__ __forceinline__ float sbyte_f(uint32_t w, int n) { return (float)(int8_t)(w >> (8 * n)); }              // byte n of w
__device__ __forceinline__ float snib_f(uint32_t w, int n) { return (float)((int32_t)(w << (28 - 4 * n)) >> 28); }   // nibble n of w
// one word of int8 codes (4) -> two words; one word of int4 codes (8) -> four words
template <int KT>
__device__ __forceinline__ void widen_int8(uint32_t w, uint32_t& o0, uint32_t& o1) {
  o0 = pack16<KT>(sbyte_f(w, 0), sbyte_f(w, 1));
  o1 = pack16<KT>(sbyte_f(w, 2), sbyte_f(w, 3));
}
template <int KT>
__device__ __forceinline__ u32x4 widen_int4(uint32_t w) {
  return u32x4{pack16<KT>(snib_f(w, 0), snib_f(w, 1)), pack16<KT>(snib_f(w, 2), snib_f(w, 3)),
               pack16<KT>(snib_f(w, 4), snib_f(w, 5)), pack16<KT>(snib_f(w, 6), snib_f(w, 7))};
}

// M: F_BF16 / F_F16 (list F; the element type is KT's) or Q_INT8 / Q_INT4 (list Q).  NCB: blocks of 16 columns, the first
// of them column c0 of the chunk's a.cq * a.G; a column is one (query token, head of the group) pair, query-major.
// n_list: entries the launch's last token sees (list F: its earlier tokens see fewer); n_walk: those of them that one of
// these columns sees.
// Code rows (list Q) are fetched as they are stored (16-byte pieces, consecutive lanes along a row), and half a tile at
// a time is widened to 16-bit values into the free upper half of the wave's tile buffer, in the layout the
// full-precision rows arrive in, where the same operand reads pick it up.  Scales stay outside the products: a K row's
// scale multiplies its logits (per 32-element group: one product per group), a V row's scale its weights.
// What becomes of the logits: not kept; scaled, in a.xs by query token; one token's, unscaled, in the LDS as far as it goes
// (k_attn_step); one token's, unscaled, in memory (k_attn_tiered)
enum Logits : int { LOG_NONE = 0, LOG_XS = 1, LOG_STEP = 2, LOG_CALL = 3 };
template <int D, int KT, Mode M, int NCB, int LOG>
__device__ __forceinline__ void attn_wave_mfma(const AttnArgs& a, const WaveLds& w, int b, int c0, int kvh, int lane,
                                               int tile0, int tstride, int n_list, int n_walk, const int* loc_list, int xcol0,
                                               f32x4 (&o)[NCB][D / 16], float (&m_run)[NCB], float (&l_run)[NCB]) {
  static_assert(KT == KT_BF16 || KT == KT_F16, "16-bit operands");
  static_assert(D % 64 == 0, "head_dim in whole 128-byte row halves");
  constexpr bool IS_Q = (M == Q_INT8 || M == Q_INT4);
  constexpr bool ONE = LOG == LOG_STEP || LOG == LOG_CALL;      // one query token: many tiles per wave, few columns
  constexpr int RB = 2 * D;                    // bytes per row as the matrix cores read it
  constexpr int TR = 8192 / RB;                // rows per tile: 8 KB
  constexpr int NRB = TR / 16, NTV = TR / 32;  // 16-entry blocks (logits), 32-entry steps (output)
  constexpr int KU = RB / 128;                 // 1 KB pieces per batch of 8 rows (operand layout)
  constexpr int NKS = D / 32, NDB = D / 16;    // instructions deep (logits), output column blocks
  constexpr int PB = 1024;
  constexpr int CRB = !IS_Q ? RB : (M == Q_INT8 ? D : D / 2);   // bytes per row as fetched
  constexpr int NP = TR * CRB / PB, NPH = NP / 2;               // 1 KB pieces per tile, K or V; of half a tile
  constexpr int LPR = CRB / 16, RPP = 64 / LPR;                 // list Q: lanes per row, rows per piece
  constexpr int SCD = (M == Q_INT8) ? 1 : (M == Q_INT4) ? D / 64 : 0;   // dwords of scales per row
  constexpr int HR = TR / 2;                                    // rows widened at a time (list Q)
  constexpr uint32_t SCR = IS_Q ? HR * RB : 0;                  // where the widened half tile sits
  static_assert(NP >= 2 && (!IS_Q || TR * CRB <= HR * RB), "two halves; code rows leave the upper half of the buffer free");
  const int g = lane >> 3, r = lane & 7;       // F fetch side: row of a batch, piece of the row's 128 bytes
  const int n = lane & 15, kb = lane >> 4;     // operand side

  __amdgpu_buffer_rsrc_t rk, rvv, rsk, rsv;
  if constexpr (!IS_Q) {
    const size_t off = (size_t)(b * a.Hkv + kvh) * a.capF * RB;
    rk = make_rsrc(a.fpK + off, (uint32_t)a.capF * RB); rvv = make_rsrc(a.fpV + off, (uint32_t)a.capF * RB);
    rsk = rk; rsv = rvv;
  } else {
    const size_t rows = (size_t)(b * a.Hkv + kvh) * a.cap2;
    rk = make_rsrc(a.c2K + rows * a.cb, (uint32_t)a.cap2 * a.cb); rvv = make_rsrc(a.c2V + rows * a.cb, (uint32_t)a.cap2 * a.cb);
    rsk = make_rsrc(a.s2K + rows * a.sb, (uint32_t)a.cap2 * a.sb); rsv = make_rsrc(a.s2V + rows * a.sb, (uint32_t)a.cap2 * a.sb);
  }
  const __amdgpu_buffer_rsrc_t rl = make_rsrc(loc_list, (uint32_t)a.Nmax * 4u);
  if (tile0 * TR >= n_walk) return;

  auto issue_loc = [&](int par, int tile) {
    if (TR == 64 || lane < TR) dma<4>(rl, w.lt + par * (TR * 4), (uint32_t)(tile * TR + lane) * 4u, 0);
  };
  // the first tile's slot list before anything else (requests are served in the order they were made)
  issue_loc(0, tile0);

  // F fetch side.  Batch i holds entries 8*i + g; its K rows are rotated by 2*(g/2) + (i & 1) pieces, its V rows by g & 6.
  const uint32_t kcol0 = (uint32_t)((r + 2 * (g >> 1)) & 7) * 16u, kcol1 = (uint32_t)((r + 2 * (g >> 1) + 1) & 7) * 16u;
  const uint32_t vcol = (uint32_t)((r + (g & 6)) & 7) * 16u;
  // operand side.  Logits: lane (n, kb) reads piece 4*ks + kb of entry 16*rb + n, which is row n & 7 of batch
  // 2*rb + n/8; one address per parity of ks, the rest are immediates.
  uint32_t k_rd[2];
  {
    const int ii = n >> 3, gg = n & 7, rot = 2 * (gg >> 1) + ii;
#pragma unroll
    for (int par = 0; par < 2; ++par)
      k_rd[par] = w.ta + SCR + (uint32_t)(ii * KU * PB) + (uint32_t)(8 * gg + ((4 * par + kb - rot) & 7)) * 16u;
  }
  // Output: in the 16 lanes of block kb, lane 4*jj + q points at elements 4*q .. 4*q+3 of column block db of entry
  // 16*rb + 4*kb + jj (row 4*(kb & 1) + jj of batch 2*rb + kb/2); one address per db & 3
  uint32_t v_rd[4];
  {
    const int jj = (lane >> 2) & 3, qq = lane & 3, ii = kb >> 1, gg = 4 * (kb & 1) + jj;
#pragma unroll
    for (int dl = 0; dl < 4; ++dl)
      v_rd[dl] = w.ta + SCR + (uint32_t)(ii * KU * PB) + (uint32_t)(8 * gg + ((2 * dl - (gg & 6)) & 7) + (qq >> 1)) * 16u + (uint32_t)(qq & 1) * 8u;
  }

  // The columns' query vectors, right operand of the logits: fetched like K rows through the tile buffer, where they arrive
  // with the slot list, and read from there as K operands are.  A column past the last repeats the last one: its products
  // are then numbers wherever a real column's are (zeros times an infinite key element would not be).
  // Direct-to-LDS loads want the alignment that the cache's own rows have; queries that begin elsewhere come by plain loads.
  int n_seen[NCB];                             // list entries the column's query may see (the chunk's later tokens are cut off list F)
  size_t xrow[NCB];                            // LOG: where the column's logits go
  bool live[NCB];
  u32x4 qreg[NCB][NKS];
  const bool q_aligned = ((uintptr_t)a.q & 15) == 0;
  {
    const int ncol = ONE ? a.G : a.cq * a.G;
    const char* qb = (const char*)a.q + (size_t)b * a.q_bs * RB;
    const float inv_g = ONE ? 0.f : 1.0f / (float)a.G;
    auto q_row = [&](int col) {                  // byte offset of a column's query vector
      col = col < ncol ? col : ncol - 1;
      const int jq = ONE ? 0 : small_div(col, inv_g);
      return (uint32_t)(jq * a.Hq + kvh * a.G + (col - jq * a.G)) * (uint32_t)RB;
    };
    if (q_aligned) {
      const __amdgpu_buffer_rsrc_t rq = make_rsrc(qb, (uint32_t)((ONE ? 1 : a.cq) * a.Hq) * RB);
#pragma unroll
      for (int i = 0; i < 2 * NCB; ++i) {
        const uint32_t off = q_row(c0 + 8 * i + g) + ((i & 1) ? kcol1 : kcol0);
#pragma unroll
        for (int j = 0; j < KU; ++j) dma<16>(rq, w.t + (i * KU + j) * PB, off + (uint32_t)j * 128u, 0);
      }
    } else {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const char* src = qb + q_row(c0 + 16 * cb + n) + 16 * kb;
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) qreg[cb][ks] = ((const PackedU32x4*)(src + 64 * ks))->v;
      }
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int col = c0 + 16 * cb + n;
      const int jq = ONE ? 0 : small_div(col, inv_g);
      live[cb] = col < ncol;
      n_seen[cb] = ONE || IS_Q || !live[cb] ? n_list : n_list - (a.cq - 1 - jq);
      if constexpr (LOG == LOG_XS) xrow[cb] = live[cb] ? xs_at(a, b * a.cq + jq, kvh * a.G + (col - jq * a.G), xcol0 + 4 * kb) : 0;
    }
  }
  // list Q: the lane's piece of a code row is widened and stored where the operand reads expect it.  Piece sl of a
  // half tile holds the half's entries RPP*sl + lane/LPR; the lane's 16 bytes are CPL 16-byte pieces of the wide row.
  constexpr int CPL = IS_Q ? RB / CRB : 1;
  auto wide_addr = [&](int sl, int k, bool v_side) -> uint32_t {
    const int el = RPP * sl + lane / LPR, i = el >> 3, gg = el & 7, cc = (lane % LPR) * CPL + k;
    const int rot = v_side ? (gg & 6) : 2 * (gg >> 1) + (i & 1);
    return w.ta + SCR + (uint32_t)((i * KU + (cc >> 3)) * PB) + (uint32_t)(8 * gg + (((cc & 7) - rot) & 7)) * 16u;
  };
  auto widen = [&](const u32x4 (&cu)[NPH], bool v_side) {
#pragma unroll
    for (int sl = 0; sl < NPH; ++sl) {
      if constexpr (M == Q_INT8) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          uint32_t w0, w1, w2, w3;
          widen_int8<KT>(elem(cu[sl], 2 * k), w0, w1);
          widen_int8<KT>(elem(cu[sl], 2 * k + 1), w2, w3);
          lds_wr128<0>(wide_addr(sl, k, v_side), u32x4{w0, w1, w2, w3});
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) lds_wr128<0>(wide_addr(sl, k, v_side), widen_int4<KT>(elem(cu[sl], k)));
      }
    }
  };

  constexpr int NLK = IS_Q ? NP : TR / 8;
  int lk[NLK], lrow = 0;                       // slots of the rows this lane fetches next (K side), and of entry `lane`
  auto read_locs = [&](int par, int nvalid) {
    const uint32_t base = w.lta + (uint32_t)par * (TR * 4u);
    if (nvalid < TR) {                                   // wave-uniform: a list's last tile
      if (lane >= nvalid && lane < TR) lds_wr32(base + (uint32_t)lane * 4u, 0xffffffffu);   // no row: fetches land as zeros
    }
    uint32_t t[NLK], me = 0;
    if constexpr (!IS_Q) {
      static_for<NLK>([&](auto ic) { constexpr int i = decltype(ic)::value; t[i] = lds_rd32<i * 32>(base + (uint32_t)g * 4u); });
    } else {
      static_for<NP>([&](auto ic) { constexpr int i = decltype(ic)::value; t[i] = lds_rd32<i * RPP * 4>(base + (uint32_t)(lane / LPR) * 4u); });
      me = lds_rd32<0>(base + (uint32_t)(lane & (TR - 1)) * 4u);
    }
    lds_wait(); tie(t); tie(me);
#pragma unroll
    for (int i = 0; i < NLK; ++i) lk[i] = (int)t[i];
    lrow = (int)me;
  };
  auto issue_scales = [&]() {                            // K scales, then V scales, of the entry `lane`
    if (TR == 64 || lane < TR) {
#pragma unroll
      for (int j = 0; j < SCD; ++j) dma<4>(rsk, w.sk + j * (TR * 4), (uint32_t)lrow * (uint32_t)a.sb + j * 4u, 0);
#pragma unroll
      for (int j = 0; j < SCD; ++j) dma<4>(rsv, w.sv + j * (TR * 4), (uint32_t)lrow * (uint32_t)a.sb + j * 4u, 0);
    }
  };
  auto issue_k_piece = [&](int s) {
    if constexpr (!IS_Q) {                               // (batch s / KU, row half s % KU)
      const int i = s / KU, j = s % KU;
      dma<16>(rk, w.t + s * PB, (uint32_t)lk[i] * (uint32_t)RB + (uint32_t)j * 128u + ((i & 1) ? kcol1 : kcol0), 1);
    } else {
      dma<16>(rk, w.t + s * PB, (uint32_t)lk[s] * (uint32_t)CRB + (uint32_t)(lane % LPR) * 16u, 1);
    }
  };

  wait_vm<0>();                                          // the list and the query vectors are in
  read_locs(0, n_walk - tile0 * TR);
  if (q_aligned) {
    static_for<NCB>([&](auto cc) {
      constexpr int cb = decltype(cc)::value;
      static_for<NKS>([&](auto kc) { constexpr int ks = decltype(kc)::value; qreg[cb][ks] = lds_rd128<(2 * cb * KU + (ks >> 1)) * PB>(k_rd[ks & 1] - SCR); });
    });
    lds_wait();
  }
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) tie(qreg[cb]);
  issue_loc(1, tile0 + tstride);
  issue_scales();
#pragma unroll
  for (int s = 0; s < NP; ++s) issue_k_piece(s);
  // the pair's first wave leaves the operand as it is for the score launch, which then reads it in lane order
  if (LOG == LOG_NONE && !IS_Q && tile0 == 0) {
    const int blocks = (a.cq * a.G + 15) / 16;
    u32x4* pk = (u32x4*)a.xs + ((size_t)(b * a.Hkv + kvh) * blocks + c0 / 16) * (NKS * 64) + lane;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb)
      if (c0 / 16 + cb < blocks) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) pk[(cb * NKS + ks) * 64] = qreg[cb][ks];
      }
  }

  int par = 1;                                           // LDS half that holds the next tile's slot list
  auto tile_body = [&](int tile, auto more_c) {
    constexpr bool MORE = decltype(more_c)::value;
    constexpr int X = MORE ? 1 : 0;
    __builtin_amdgcn_s_setprio(MORE ? 3 : 1);
    int lv[NLK];                                         // this tile's V rows are fetched from the same slots
#pragma unroll
    for (int i = 0; i < NLK; ++i) lv[i] = lk[i];
    auto issue_v_piece = [&](int v) {
      if constexpr (!IS_Q) {
        const int i = v / KU, j = v % KU;
        dma<16>(rvv, w.t + v * PB, (uint32_t)lv[i] * (uint32_t)RB + (uint32_t)j * 128u + vcol, 1);
      } else {
        dma<16>(rvv, w.t + v * PB, (uint32_t)lv[v] * (uint32_t)CRB + (uint32_t)(lane % LPR) * 16u, 1);
      }
    };
    if constexpr (MORE) {
      wait_vm<2 * SCD + NP>();                           // younger than the next list: this tile's scales and K pieces
      read_locs(par, n_walk - (tile + tstride) * TR);
      issue_loc(par ^ 1, tile + 2 * tstride);
    }
    // -- logits, 16 entries at a time
    f32x4 c[NCB][NRB];
    auto logits_of = [&](auto rc, const u32x4 (&ka)[NKS]) {    // rc: the 16-entry block
      constexpr int rb = decltype(rc)::value;
      if constexpr (M == Q_INT4) {
        // one product per scale group; the four entries' scales of dword ks/2, half ks & 1
        u32x4 sc[SCD];
        static_for<SCD>([&](auto jc) { constexpr int j = decltype(jc)::value; sc[j] = lds_rd128<j * (TR * 4) + rb * 64>(w.ska + (uint32_t)kb * 16u); });
        lds_wait(); tie(sc);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks) {
            f32x4 part = {0.f, 0.f, 0.f, 0.f};
            if constexpr (ONE) {
              const u32x4 x = ka[ks], y = qreg[cb][ks];
              const f32x4 lo = mfma_16x16x16<KT>(u32x2{x.x, x.y}, u32x2{y.x, y.y}, part), hi = mfma_16x16x16<KT>(u32x2{x.z, x.w}, u32x2{y.z, y.w}, part);
#pragma unroll
              for (int j = 0; j < 4; ++j) part[j] = lo[j] + hi[j];
            } else part = mfma_16x16x32<KT>(ka[ks], qreg[cb][ks], part);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j] = fmaf(half_of(elem(sc[ks >> 1], j), ks & 1), part[j], acc[j]);
          }
          c[cb][rb] = acc;
        }
      } else {
        if constexpr (ONE) {
          // A quarter of the elements at a time, then added in pairs (a chain of four is 1.5 times as far off, dot products on the
          // vector ALUs about as far; 128 elements, one of them large: rms 3.3e-6, 2.2e-6, 2.2e-6)
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) {
            f32x4 part[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
              if constexpr (NKS == 4) part[i] = mfma_16x16x32<KT>(ka[i], qreg[cb][i], zero);
              else {                                     // the first or last four of every lane's eight elements
                const u32x4 x = ka[i >> 1], y = qreg[cb][i >> 1];
                part[i] = (i & 1) ? mfma_16x16x16<KT>(u32x2{x.z, x.w}, u32x2{y.z, y.w}, zero) : mfma_16x16x16<KT>(u32x2{x.x, x.y}, u32x2{y.x, y.y}, zero);
              }
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) c[cb][rb][j] = (part[0][j] + part[1][j]) + (part[2][j] + part[3][j]);
          }
        } else {
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb) c[cb][rb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) c[cb][rb] = mfma_16x16x32<KT>(ka[ks], qreg[cb][ks], c[cb][rb]);
        }
        if constexpr (M == Q_INT8) {
          u32x4 sc = lds_rd128<rb * 64>(w.ska + (uint32_t)kb * 16u);
          lds_wait(); tie(sc);
#pragma unroll
          for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int j = 0; j < 4; ++j) c[cb][rb][j] *= elem_f(sc, j);
        }
      }
    };
    if constexpr (!IS_Q) {
      // the K rows of 16 entries that have been read are replaced by V pieces
      u32x4 ka[2][NKS];
      auto read_k = [&](auto rc, u32x4 (&dst)[NKS]) {
        constexpr int rb = decltype(rc)::value;
        // younger than these K pieces: the later K pieces, this period's list fetch, the V pieces so far
        wait_vm<NP - 2 * KU + X>();
        static_for<NKS>([&](auto kc) {
          constexpr int ks = decltype(kc)::value;
          dst[ks] = lds_rd128<(rb * 2 * KU + (ks >> 1)) * PB>(k_rd[ks & 1]);
        });
      };
      read_k(std::integral_constant<int, 0>{}, ka[0]);
      static_for<NRB>([&](auto rc) {
        constexpr int rb = decltype(rc)::value;
        lds_wait(); tie(ka[rb & 1]);
#pragma unroll
        for (int v = 2 * rb * KU; v < (2 * rb + 2) * KU; ++v) issue_v_piece(v);
        if constexpr (rb + 1 < NRB) read_k(std::integral_constant<int, (rb + 1 < NRB ? rb + 1 : NRB - 1)>{}, ka[(rb + 1) & 1]);
        logits_of(rc, ka[rb & 1]);
      });
    } else {
      // half a tile of code rows is widened, then replaced by V pieces
      static_for<2>([&](auto hc) {
        constexpr int hf = decltype(hc)::value;
        // younger than this half's K pieces: the other half's, this period's list fetch, the V pieces so far
        wait_vm<NP - NPH + X>();
        u32x4 cu[NPH];
        static_for<NPH>([&](auto sc) { constexpr int sl = decltype(sc)::value; cu[sl] = lds_rd128<(hf * NPH + sl) * PB>(w.ta + (uint32_t)lane * 16u); });
        lds_wait(); tie(cu);
#pragma unroll
        for (int v = hf * NPH; v < (hf + 1) * NPH; ++v) issue_v_piece(v);
        widen(cu, false);
        static_for<NRB / 2>([&](auto rlc) {
          constexpr int rl2 = decltype(rlc)::value;
          u32x4 ka[NKS];
          static_for<NKS>([&](auto kc) {
            constexpr int ks = decltype(kc)::value;
            ka[ks] = lds_rd128<(rl2 * 2 * KU + (ks >> 1)) * PB>(k_rd[ks & 1]);
          });
          lds_wait(); tie(ka);
          logits_of(std::integral_constant<int, NRB / 2 * hf + rl2>{}, ka);
        });
      });
    }
    // -- online softmax: the lane has entries 16*rb + 4*kb + j of its column
    // One token in binary16, whose terms end at 2^-24: the tile's weights enter the product relative to the column's largest
    // (the power of two above it), and list Q's V scales relative to the tile's largest, and the tile's sum gets both back:
    // weights down to 1 / 8192 of the tile's largest are whole in the three terms, whatever the values' magnitude and wherever
    // the tile lies below the running maximum.  A tile that has smaller ones adds what the terms leave of them by itself.
    // (All times 2^14, as a chunk's: values of 1e-4 in int8 rows were 3.4e-6 from 64 bits, as any others now 3.0e-7, and beside a
    // first row with all of the attention but e^-24 and a value of zero outputs were 1.2e-3 off.)
    constexpr bool REL = ONE && KT == KT_F16;
    uint32_t rel = 0;                                    // REL: that power of two, as bits
    int wide = 0;                                        // ... wave-uniform: smaller weights; 2: ones that take a second round
    float p[NCB][NRB][4];
    {
      const int e0 = tile * TR + 4 * kb;
      const bool edge = (tile + 1) * TR > n_list - (ONE || IS_Q ? 0 : a.cq - 1);   // wave-uniform: some column does not see the whole tile
      // A chunk's binary16 code rows: a weight times its V row's scale has to stay in binary16's range.  Where the tile has a
      // scale beyond what the shift leaves room for (V of some 26 and more in an int4 group, 480 in an int8 row), such an entry
      // counts with the logit of its scaled weight in the running reference, which is then above the largest logit: any
      // reference does, the statistics are merged relative to it.
      constexpr bool BOUND = IS_Q && KT == KT_F16 && !ONE;
      bool big = false;                                  // wave-uniform
      if constexpr (BOUND) {
        uint32_t sv[SCD];
        static_for<SCD>([&](auto jc) { constexpr int j = decltype(jc)::value; sv[j] = lds_rd32<j * (TR * 4)>(w.sva + (uint32_t)(lane & (TR - 1)) * 4u); });
        lds_wait(); tie(sv);
        float s = 0.f;
#pragma unroll
        for (int j = 0; j < SCD; ++j) s = fmaxf(s, M == Q_INT8 ? __builtin_bit_cast(float, sv[j]) : fmaxf(half_of(sv[j], 0), half_of(sv[j], 1)));
        big = __builtin_amdgcn_ballot_w64(s > PSplit<KT>::SCALE_MAX) != 0;
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        float mx = -INFINITY;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int j = 0; j < 4; ++j) p[cb][rb][j] = c[cb][rb][j] * a.softmax_scale;
        float least = INFINITY;                          // REL: the lane's smallest logit but masked ones
        if (edge) {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const bool seen = e0 + 16 * rb + j < n_seen[cb];
              if constexpr (REL) least = fminf(least, seen ? p[cb][rb][j] : INFINITY);
              p[cb][rb][j] = seen ? p[cb][rb][j] : -INFINITY;
            }
        } else if constexpr (REL) {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int j = 0; j < 4; ++j) least = fminf(least, p[cb][rb][j]);
        }
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int j = 0; j < 4; ++j) mx = fmaxf(mx, p[cb][rb][j]);
        if constexpr (BOUND) {
          if (big)
            static_for<NRB>([&](auto rc) {
              constexpr int rb = decltype(rc)::value;
              u32x4 sv[SCD];
              static_for<SCD>([&](auto jc) { constexpr int i = decltype(jc)::value; sv[i] = lds_rd128<i * (TR * 4) + rb * 64>(w.sva + (uint32_t)kb * 16u); });
              lds_wait(); tie(sv);
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                float s = PSplit<KT>::SCALE_MAX;
#pragma unroll
                for (int i = 0; i < SCD; ++i) s = fmaxf(s, M == Q_INT8 ? elem_f(sv[i], j) : fmaxf(half_of(elem(sv[i], j), 0), half_of(elem(sv[i], j), 1)));
                s = fminf(s, 65536.f);                   // (a scale is at most 65504 / 7; infinite ones stay infinite in the product)
                mx = fmaxf(mx, fmaf(__builtin_amdgcn_logf(s * (1.0f / PSplit<KT>::SCALE_MAX)), LN2, p[cb][rb][j]));
              }
            });
        }
        if constexpr (LOG == LOG_STEP) {
          const int col = xcol0 + tile * TR + 4 * kb;
          if (live[cb]) {
            if (xcol0 + tile * TR + TR <= w.lim) {
              static_for<NRB>([&](auto rc) {
                constexpr int rb = decltype(rc)::value;
                u32x4 t;
#pragma unroll
                for (int j = 0; j < 4; ++j) { const float x = c[cb][rb][j]; t[j] = __builtin_bit_cast(uint32_t, x); }
                lds_wr128<rb * 64>(w.lga + (uint32_t)(n * w.lcap + col) * 4u, t);
              });
            } else {
              float* sp = w.sp + (size_t)n * w.sp_stride + col;
#pragma unroll
              for (int rb = 0; rb < NRB; ++rb) *(f32x4*)(sp + 16 * rb) = c[cb][rb];
            }
          }
        }
        if constexpr (LOG == LOG_CALL) {
          if (live[cb]) {
            float* sp = w.sp + (size_t)n * w.sp_stride + (xcol0 + tile * TR + 4 * kb);
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb) *(f32x4*)(sp + 16 * rb) = c[cb][rb];
          }
        }
        if constexpr (LOG == LOG_XS) {
          if (live[cb]) {
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb)
              *(f32x4*)(a.xs + xrow[cb] + (size_t)tile * TR + 16 * rb) = f32x4{p[cb][rb][0], p[cb][rb][1], p[cb][rb][2], p[cb][rb][3]};
          }
        }
        // m_run starts at -inf: corr = exp2(-inf) = 0 against zero accumulators.  A tile of which the column sees
        // nothing (an early token of a chunk, the list's last tile) leaves mn at -inf: nothing to add, nothing to rescale.
        const float mt = quad_max(mx), mn = fmaxf(m_run[cb], mt);
        const float corr = mn > -INFINITY ? __builtin_amdgcn_exp2f((m_run[cb] - mn) * LOG2E) : 1.0f;
        const float ms = mn > -INFINITY ? mn : 0.f;      // (all weights are exp2(-inf) = 0 then)
        float ps = 0.f;
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            // (one token: the product's rounding is left out of the distance to the reference; a masked entry stays one, and a
            // logit that is no number stays none)
            const float d = ONE ? (p[cb][rb][j] == -INFINITY ? -INFINITY : fmaf(c[cb][rb][j], a.softmax_scale, -ms)) : p[cb][rb][j] - ms;
            if constexpr (ONE) p[cb][rb][j] = exp_le0(d);
            else p[cb][rb][j] = __builtin_amdgcn_exp2f(fmaf(d, LOG2E, PSplit<KT>::P_SHIFT));
            ps += p[cb][rb][j];
          }
        l_run[cb] = fmaf(l_run[cb], corr, ps);
        m_run[cb] = mn;
        if constexpr (REL) {
          // (2^-64 of the running maximum: nothing the outputs could hold)
          rel = (__builtin_bit_cast(uint32_t, fmaxf(__builtin_amdgcn_exp2f((mt - ms) * LOG2E), 0x1p-64f)) & 0x7f800000u) + 0x800000u;
          // (e^9 is just below 8192; e^35 below 2^51: down to there a weight's 24 bits end within the first round's 2^-62)
          if (__builtin_amdgcn_ballot_w64(mt - least > 9.0f) != 0) wide = __builtin_amdgcn_ballot_w64(mt - least > 35.0f) != 0 ? 2 : 1;
        }
        // the output accumulators of this lane belong to columns 4*kb + j: their factors come from those columns'
        // lanes; once the maxima have settled nothing needs rescaling (x * 1.0f is exact)
        if (__builtin_amdgcn_ballot_w64(corr != 1.0f) != 0) {
          float cj[4];
#pragma unroll
          for (int j = 0; j < 4; ++j)
            cj[j] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((4 * kb + j) << 2, __builtin_bit_cast(int, corr)));
#pragma unroll
          for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int j = 0; j < 4; ++j) o[cb][db][j] *= cj[j];
        }
      }
    }
    // -- output: 32 entries per instruction; V rows that have been read are replaced by K pieces
    __builtin_amdgcn_s_setprio(MORE ? 2 : 0);
    constexpr int NT = ONE ? 3 : PSplit<KT>::N;
    // V scales of the tile: the 4 entries' of each 16-entry block (all older than the K pieces: they are in)
    u32x4 vsc[IS_Q ? SCD : 1][NRB];
    if constexpr (IS_Q) {
      static_for<SCD>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        static_for<NRB>([&](auto rc) { constexpr int rb = decltype(rc)::value; vsc[j][rb] = lds_rd128<j * (TR * 4) + rb * 64>(w.sva + (uint32_t)kb * 16u); });
      });
      lds_wait();
#pragma unroll
      for (int j = 0; j < SCD; ++j) tie(vsc[j]);
      if constexpr (MORE) issue_scales();                // both scale regions are free: the next tile's
    }
    float unit[4] = {1.f, 1.f, 1.f, 1.f};                // what the tile's sums of columns 4*kb + j are in units of
    if constexpr (REL) {
      // 2^14 / rel, and unit its inverse; list Q: over the power of two at or below the tile's largest scale as well
      float up = __builtin_bit_cast(float, 0x7f000000u + (14u << 23) - rel), down = __builtin_bit_cast(float, rel - (14u << 23));
      if constexpr (IS_Q) {
        float s = 0.f;
        if constexpr (M == Q_INT8) {
#pragma unroll
          for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
            for (int j = 0; j < 4; ++j) s = fmaxf(s, elem_f(vsc[0][rb], j));
        } else {
          u16x2 t = {0, 0};                              // (no scale is negative: their order is that of their bits)
#pragma unroll
          for (int i = 0; i < SCD; ++i)
#pragma unroll
            for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
              for (int j = 0; j < 4; ++j) t = __builtin_elementwise_max(t, __builtin_bit_cast(u16x2, elem(vsc[i][rb], j)));
          s = fmaxf(half_of(t.x, 0), half_of(t.y, 0));
        }
        // (no scale of a binary16 row but zero and infinity lies outside; an infinite one stays infinite in the product)
        const uint32_t e = __builtin_bit_cast(uint32_t, fminf(fmaxf(quad_max(s), 0x1p-40f), 0x1p20f)) & 0x7f800000u;
        up *= __builtin_bit_cast(float, 0x7f000000u - e);
        down *= __builtin_bit_cast(float, e);
      }
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
        for (int j = 0; j < 4; ++j) p[0][rb][j] *= up;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        unit[j] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((4 * kb + j) << 2, __builtin_bit_cast(int, down)));
    }
    // weights of 32 entries; list Q: times the V row's scale (of scale group gd)
    auto products = [&](auto tc, int cb, int gd, float (&pw)[2][4]) {
      constexpr int t = decltype(tc)::value;
#pragma unroll
      for (int r2 = 0; r2 < 2; ++r2)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float v = p[cb][2 * t + r2][j];
          if constexpr (M == Q_INT8) v *= elem_f(vsc[0][2 * t + r2], j);
          if constexpr (M == Q_INT4) v *= half_of(elem(vsc[gd >> 1][2 * t + r2], j), gd & 1);
          pw[r2][j] = v;
        }
    };
    // ... as operand terms
    auto terms = [&](float (&pw)[2][4], u32x4 (&pt)[NT]) {
      uint32_t s0[NT], s1[NT], s2[NT], s3[NT];
      split_pair<KT, NT>(pw[0][0], pw[0][1], s0);
      split_pair<KT, NT>(pw[0][2], pw[0][3], s1);
      split_pair<KT, NT>(pw[1][0], pw[1][1], s2);
      split_pair<KT, NT>(pw[1][2], pw[1][3], s3);
#pragma unroll
      for (int i = 0; i < NT; ++i) pt[i] = u32x4{s0[i], s1[i], s2[i], s3[i]};
    };
    // list Q: half a tile of V codes (hf) is widened, its place refilled with the next tile's K pieces
    auto widen_v = [&](auto hc) {
      constexpr int hf = decltype(hc)::value;
      // younger than this half's V pieces: the other half's, the next tile's scales, the K pieces issued after the first half
      wait_vm<NPH * (1 - hf) + X * (2 * SCD + hf * NPH)>();
      u32x4 cu[NPH];
      static_for<NPH>([&](auto sc) { constexpr int sl = decltype(sc)::value; cu[sl] = lds_rd128<(hf * NPH + sl) * PB>(w.ta + (uint32_t)lane * 16u); });
      lds_wait(); tie(cu);
      if constexpr (MORE) {
#pragma unroll
        for (int s = hf * NPH; s < (hf + 1) * NPH; ++s) issue_k_piece(s);
      }
      widen(cu, true);
    };
    f32x4 sum[ONE ? NDB : 1];                            // one token: the tile's own sum, of many tiles per wave
#pragma unroll
    for (int db = 0; db < (ONE ? NDB : 1); ++db) sum[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    static_for<NTV>([&](auto tc) {
      constexpr int t = decltype(tc)::value;
      constexpr int NPV = NP / NTV;                      // V pieces of this step
      u32x2 vv[2][NDB];
      auto read_vv = [&](auto rc, auto bc) {             // 16 entries (rc of the step), which sit bc 16-row blocks into their area
        constexpr int r2 = decltype(rc)::value, rb = decltype(bc)::value;
        static_for<NDB>([&](auto dc) {
          constexpr int db = decltype(dc)::value;
          vv[r2][db] = lds_rd64_tr16<(rb * 2 * KU + (db >> 2)) * PB>(v_rd[db & 3]);
        });
      };
      constexpr std::integral_constant<int, 0> I0{};
      constexpr std::integral_constant<int, 1> I1{};
      if constexpr (!IS_Q) {
        // younger than this step's V pieces: the later steps', the next tile's K pieces so far
        wait_vm<NPV * (NTV - 1 - t) + X * t * NPV>();
        read_vv(I0, std::integral_constant<int, 2 * t>{});
        read_vv(I1, std::integral_constant<int, 2 * t + 1>{});
        lds_wait(); tie(vv[0]); tie(vv[1]);
        if constexpr (MORE) {
#pragma unroll
          for (int s = t * NPV; s < (t + 1) * NPV; ++s) issue_k_piece(s);
        }
      } else if constexpr (NTV == 2) {                   // a half tile is a step
        widen_v(tc);
        read_vv(I0, I0);
        read_vv(I1, I1);
        lds_wait(); tie(vv[0]); tie(vv[1]);
      } else {                                           // a half tile is 16 entries
        widen_v(I0);
        read_vv(I0, I0);
        lds_wait(); tie(vv[0]);
        widen_v(I1);
        read_vv(I1, I0);
        lds_wait(); tie(vv[1]);
      }
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        u32x4 pt[NT];
        float pw[2][4];
        if constexpr (M != Q_INT4) { products(tc, cb, 0, pw); terms(pw, pt); }
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          if constexpr (M == Q_INT4) { if (db % 2 == 0) { products(tc, cb, db / 2, pw); terms(pw, pt); } }
          const u32x4 vb = u32x4{vv[0][db].x, vv[0][db].y, vv[1][db].x, vv[1][db].y};
          if constexpr (ONE) {
            // small terms first, and one addition to the running output per tile
#pragma unroll
            for (int i = NT - 1; i >= 0; --i) sum[db] = mfma_16x16x32<KT>(pt[i], vb, sum[db]);
            if constexpr (t + 1 == NTV) {
#pragma unroll
              for (int j = 0; j < 4; ++j) o[cb][db][j] = fmaf(sum[db][j], unit[j], o[cb][db][j]);
            }
          } else {
#pragma unroll
            for (int i = NT - 1; i >= 0; --i) o[cb][db] = mfma_16x16x32<KT>(pt[i], vb, o[cb][db]);
          }
        }
        if constexpr (REL) {
          if (wide > 0) {
            // what the terms leave (below 2^-24), times 2^38, and what that leaves once more
            constexpr int GDB = M == Q_INT4 ? 2 : NDB;   // columns of output with the same weights
#pragma unroll
            for (int g0 = 0; g0 < NDB; g0 += GDB) {
              float f = 1.0f;
              products(tc, cb, g0 / 2, pw);
              terms(pw, pt);
              for (int k = 0; k < wide; ++k) {
                f *= 0x1p-38f;
#pragma unroll
                for (int r2 = 0; r2 < 2; ++r2)
#pragma unroll
                  for (int j = 0; j < 4; ++j) pw[r2][j] *= 0x1p38f;
                terms(pw, pt);
#pragma unroll
                for (int db = g0; db < g0 + GDB; ++db) {
                  const u32x4 vb = u32x4{vv[0][db].x, vv[0][db].y, vv[1][db].x, vv[1][db].y};
                  f32x4 rest = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                  for (int i = NT - 1; i >= 0; --i) rest = mfma_16x16x32<KT>(pt[i], vb, rest);
#pragma unroll
                  for (int j = 0; j < 4; ++j) o[cb][db][j] = fmaf(rest[j], unit[j] * f, o[cb][db][j]);
                }
              }
            }
          }
        }
      }
    });
    par ^= 1;
  };

  int tile = tile0;
  for (; (tile + tstride) * TR < n_walk; tile += tstride) tile_body(tile, std::true_type{});
  tile_body(tile, std::false_type{});

  if constexpr (PSplit<KT>::P_SHIFT != 0.f && !ONE) {
    const float back = __builtin_amdgcn_exp2f(-PSplit<KT>::P_SHIFT);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      l_run[cb] *= back;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int j = 0; j < 4; ++j) o[cb][db][j] *= back;
    }
  }
}

// One token's result of a wave into LDS: lane (n, kb) has the statistics of head n and the outputs of heads 4*kb + j, element 16*db + n
template <int D, int G>
__device__ __forceinline__ void park_one(const f32x4 (&om)[D / 16], float m, float l, int lane, float* o, float* ml) {
  const float ls = quad_sum(l);
  if (lane < G) { ml[lane] = m; ml[8 + lane] = ls; }
#pragma unroll
  for (int db = 0; db < D / 16; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int h = 4 * (lane >> 4) + j;
      if (h < G) o[h * D + 16 * db + (lane & 15)] = om[db][j];
    }
}

// The same of a wave on the vector ALUs: the row groups are summed, and the per-lane denominators
template <int D, int G, int EV, int LPRV>
__device__ __forceinline__ void park_rows(const float (&o)[G][EV], int lane, float* my_o) {
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float t[RowSum<EV, LPRV>::N];
    row_sum<EV, LPRV>(o[h], lane, t);
#pragma unroll
    for (int k = 0; k < RowSum<EV, LPRV>::N; ++k) my_o[h * D + row_sum_elem<EV, LPRV>(lane, k)] = t[k];
  }
}
template <int G>
__device__ __forceinline__ void park_stats(const float (&m_run)[G], const float (&l_lane)[G], int lane, float* ml) {
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float ls = wave_sum(l_lane[h]);
    if (lane == 0) { ml[h] = m_run[h]; ml[8 + h] = ls; }
  }
}

// Whether a wave's outputs are all finite, in every lane (the padding columns' are those of the last head)
template <int D>
__device__ __forceinline__ bool finite_one(const f32x4 (&om)[D / 16]) {
  float z[4] = {0.f, 0.f, 0.f, 0.f};                     // (infinity times zero is no number, as no number is)
#pragma unroll
  for (int db = 0; db < D / 16; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j) z[j] = fmaf(om[db][j], 0.f, z[j]);
  return __builtin_amdgcn_ballot_w64((z[0] + z[1]) + (z[2] + z[3]) != 0.f) == 0;
}

// One token's outputs of a wave once more, a product at a time: on the matrix cores an infinite value has no number for its
// output wherever a term of its weight is zero (the largest weight's second, for one), where weight times value is infinite.
// From the logits that the wave has left behind, its final maxima and the rows, all of it plain: a lane has D / 64 elements of
// every head, the wave its rows one after the other.  Only for waves of which some output is no finite number.
template <int D, int G, int KT, Mode M, int LOG>
__device__ __forceinline__ void outputs_plain(const AttnArgs& a, const WaveLds& w, int b, int kvh, int lane, int tile0, int tstride,
                                              int n_list, const int* loc_list, int xcol0, float m, float* o) {
  constexpr bool IS_Q = (M == Q_INT8 || M == Q_INT4);
  constexpr int TR = 4096 / D, EPL = D / 64;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");  // the logits, which other lanes have stored
  lds_wait();
  const size_t pair = (size_t)b * a.Hkv + kvh;
  const int el = lane * EPL;
  float acc[G][EPL], ms[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const float mh = rdlane(m, h);
    ms[h] = mh > -INFINITY ? mh : 0.f;
#pragma unroll
    for (int k = 0; k < EPL; ++k) acc[h][k] = 0.f;
  }
  for (int tile = tile0; tile * TR < n_list; tile += tstride) {
    const bool in_lds = LOG == LOG_STEP && xcol0 + tile * TR + TR <= w.lim;
    for (int i = tile * TR; i < tile * TR + TR && i < n_list; ++i) {
      const int slot = loc_list[i], col = xcol0 + i;
      float v[EPL], sc = 1.f;
#pragma unroll
      for (int k = 0; k < EPL; ++k) v[k] = 0.f;          // (no row: zeros, as fetched by the tile)
      if ((uint32_t)slot < (uint32_t)(IS_Q ? a.cap2 : a.capF)) {
        if constexpr (!IS_Q) {
          const uint16_t* row = (const uint16_t*)(a.fpV + (pair * a.capF + slot) * (2 * D)) + el;
#pragma unroll
          for (int k = 0; k < EPL; ++k) v[k] = KT == KT_BF16 ? bf_lo(row[k]) : half_of(row[k], 0);
        } else {
          const size_t r = pair * a.cap2 + slot;
          const uint8_t* codes = (const uint8_t*)a.c2V + r * a.cb;
#pragma unroll
          for (int k = 0; k < EPL; ++k) v[k] = M == Q_INT8 ? sbyte_f(codes[el + k], 0) : snib_f(codes[(el + k) / 2], (el + k) & 1);
          sc = M == Q_INT8 ? *(const float*)(a.s2V + r * a.sb) : half_of(((const uint16_t*)(a.s2V + r * a.sb))[el / 32], 0);
        }
      }
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float x;
        if (in_lds) {
          uint32_t t = lds_rd32<0>(w.lga + (uint32_t)(h * w.lcap + col) * 4u);
          lds_wait(); tie(t);
          x = __builtin_bit_cast(float, t);
        } else x = w.sp[(size_t)h * w.sp_stride + col];
        float p = exp_le0(fmaf(x, a.softmax_scale, -ms[h]));
        if constexpr (IS_Q) p *= sc;
#pragma unroll
        for (int k = 0; k < EPL; ++k) acc[h][k] = fmaf(p, v[k], acc[h][k]);
      }
    }
  }
#pragma unroll
  for (int h = 0; h < G; ++h)
#pragma unroll
    for (int k = 0; k < EPL; ++k) o[h * D + el + k] = acc[h][k];
}

// Geometry of the split launch: rows per tile and waves per workgroup (one workgroup per compute unit).  16-bit rows: 8 KB
// tiles (32 rows of 256 bytes, 64 of 128) and eight waves, two per SIMD; 64 KB in flight per compute unit stream as fast
// as 128 KB do, and the finer tiles keep more waves busy on short lists and end closer together on long ones.  binary32
// rows: 32 rows of 256 bytes; 64 rows of 512 bytes with four waves, which large groups take in any case (their waves need
// more than half a SIMD's registers).
// Whether a split launch's waves run on the matrix cores.  us a call, vector / matrix instructions, 12 % int8 T2, head_dim 128: 28/4
// heads, 1 x 300 tokens 11.6 / 10.3, 1 x 1422 12.9 / 11.7, 1 x 16000 21.4 / 19.2, 8 x 2081 18.2 / 15.8; 64/8, 1 x 2000 13.8 / 11.8;
// 40/8, 8 x 4133 32.2 / 31.6; 10/2, 16 x 1000 12.4 / 12.2; 16/4, 30 x 700 15.4 / 14.4; but 6/2, 8 x 3000 12.5 / 12.7, 4/2, 2 x 5000
// 13.2 / 13.6, 4/4, 1 x 9000 13.7 / 14.5: with few heads the vector ALUs have little to do, and a wave's first products wait
// for the queries.  At head_dim 64 calls would be faster (28/4, 1 x 1422 12.8 / 10.8, 64/8, 4 x 4000 18.6 / 15.5), but outputs
// further from 64 bits (16/4, 1 x 2500 2.0e-7 / 2.1e-7; 12/2, 2 x 5000, int4 2.6e-7 / 2.75e-7; 64/8, 2 x 3000 2.2e-7 / 2.25e-7).
// Outputs against 64 bits at head_dim 128: 28/4, 1 x 1422 2.5e-7 / 2.3e-7; 40/8, 8 x 4133 3.2e-7 / 2.5e-7; binary16, 28/4,
// 2 x 9000, int4 3.4e-7 / 3.0e-7; 10/2, 3 x 300, int4 2.1e-7 / 1.9e-7.
constexpr bool split_on_matrix(int D, int G, int q_es) { return q_es == 2 && D == 128 && G >= 4; }
template <int D, int G, int KT>
struct KernelGeo {
  static constexpr bool MC = split_on_matrix(D, G, KT == KT_F32 ? 4 : 2);
  static constexpr Mode MF = KT == KT_BF16 ? F_BF16 : KT == KT_F16 ? F_F16 : F_F32;
  static constexpr int RB = Geo<D, MF>::RB;
  static constexpr int TR = RB == 256 ? 32 : 64, TILE = TR * RB;
  static constexpr int NW = KT == KT_F32 && (G > 5 || RB > 256) ? 4 : 8;
  static constexpr int EV = Geo<D, MF, TR>::EV;
  static constexpr int LPRV = Geo<D, MF, TR>::LPRV;
};
constexpr int split_tile_rows(int D, int es) { return D * es == 256 ? 32 : 64; }
constexpr int split_waves(int D, int es, int G) { return es == 4 && (G > 5 || D * es > 256) ? 4 : 8; }

// Waves of a (sequence, kv head) pair that serve the Q list, out of nwv, for nft F tiles and nqt Q tiles: the split
// that minimises the longest wave.  A code tile moves fewer bytes than a full-precision one but costs more vector
// instructions (unpacking); it is priced QCOST_Q against QCOST_F for an F tile.  Depends on the list lengths only.
constexpr int QCOST_F = 4, QCOST_Q = 5;
__host__ __device__ inline int q_waves(int nwv, int nft, int nqt) {
  if (nqt == 0) return 0;
  if (nft == 0) return nwv;
  int best = 1, best_cost = 0x7fffffff;
  for (int n = 1; n < nwv; ++n) {
    const int cf = ((nft + (nwv - n) - 1) / (nwv - n)) * QCOST_F, cq = ((nqt + n - 1) / n) * QCOST_Q;
    const int c = cf > cq ? cf : cq;
    if (c < best_cost) { best_cost = c; best = n; }
  }
  return best;
}

template <int D, int G, int KT>
__global__ __launch_bounds__((KernelGeo<D, G, KT>::NW * 64), (KernelGeo<D, G, KT>::NW / 4)) void k_attn_tiered(const AttnArgs a) {
  using KG = KernelGeo<D, G, KT>;
  constexpr int NW = KG::NW, EV = KG::EV, LPRV = KG::LPRV, GP = GPad<G>::v, TR = KG::TR;
  constexpr int TILE_BYTES = KG::TILE, SC = (D / 64) * TR * 4;
  static_assert(G * D * 4 <= TILE_BYTES, "a wave's output partial is parked in its tile buffer");
  __shared__ __attribute__((aligned(16))) char sm_t[NW * TILE_BYTES];
  __shared__ __attribute__((aligned(16))) char sm_sc[NW * 2 * SC];
  __shared__ __attribute__((aligned(16))) char sm_lt[NW * 2 * TR * 4];
  __shared__ __attribute__((aligned(16))) float sm_p[NW * TR * GP];
  __shared__ float sm_ml[NW * 16];
  const int s = blockIdx.x, kvh = blockIdx.y;
  // The arguments come over the host link (about a microsecond): a call's sequence is blockIdx.z, so its list lengths are
  // asked for with everything else, not behind n_q, nl and B, and corrected where the launch is of another kind.
  int b = blockIdx.z, jq = 0, li = 0, nF = a.nF[b & (ATTN_ARG_SEQS - 1)], nQ = a.nQ[b & (ATTN_ARG_SEQS - 1)];
  int nwq = a.nWq[b & (ATTN_ARG_SEQS - 1)], xsb = 0;
  const int nwv = a.S * NW;
  if (a.n_q > 1 || a.nl > 1 || a.B > ATTN_ARG_SEQS || a.second) {
    // several query tokens per sequence: query jq of sequence b; it is n_q - 1 - jq positions older than the last one,
    // and those positions (the tail of list F) are not its to see
    if (a.n_q > 1) { jq = b % a.n_q; b = b / a.n_q; }
    // a whole decode step: layer li of the launch's a.nl
    else if (a.nl > 1) { li = b / a.B; b -= li * a.B; }
    if (a.second) {
      nF = a.cnt[b * CNT_N + C_NS]; nQ = 0; nwq = 0;
      xsb = ((a.cnt[b * CNT_N + C_NF] - a.trim + 63) >> 6) + ((a.cnt[b * CNT_N + C_NQ] + 63) >> 6);
    } else {
      if (a.B <= ATTN_ARG_SEQS) { nF = a.nF[b]; nQ = a.nQ[b]; nwq = a.nWq[b]; }
      else { nF = a.cnt[b * CNT_N + C_NF] - a.trim; nQ = a.cnt[b * CNT_N + C_NQ]; }
      nF -= a.n_q - 1 - jq;
      if (a.B > ATTN_ARG_SEQS || a.n_q > 1) nwq = q_waves(nwv, (nF + TR - 1) / TR, (nQ + TR - 1) / TR);
    }
  }
  const int bl = li * a.B + b;                  // entry of rows, q, logits and partials
  const int* f_loc = ((a.old_mask >> li) & 1) ? a.f_loc_old : a.f_loc;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int nft = (nF + TR - 1) / TR, nqt = (nQ + TR - 1) / TR, nwf = nwv - nwq;
  const int colq = (xsb + ((nF + 63) >> 6)) * TB;   // list Q's logits start at a 64-entry tile
  // Which wave of the pair this is.  Workgroup by workgroup, so that the waves of list Q, the last ones, sit together: a
  // compute unit that runs one list's code only keeps it in its instruction cache (14B shape 2.5 %, 7B 4 % faster than
  // dealt out over the workgroups).  With two or three workgroups the one with the Q waves would have too few bytes to
  // fetch (2 % slower at 63 x 2 pairs), and a short pair (up to four tiles per workgroup) is to have one tile per SIMD:
  // these are dealt out wave by wave.
  const int u = a.S < 4 || nft + nqt <= 4 * a.S ? wave * a.S + s : s * NW + wave;

  WaveLds w;
  w.t = sm_t + wave * TILE_BYTES;
  w.sk = sm_sc + wave * 2 * SC; w.sv = w.sk + SC; w.lt = sm_lt + wave * 2 * TR * 4;
  w.ta = lds_addr(w.t); w.ska = lds_addr(w.sk); w.sva = lds_addr(w.sv); w.lta = lds_addr(w.lt);
  w.p = (char*)(sm_p + wave * TR * GP);
  w.pa = lds_addr(w.p);
  float* my_o = (float*)w.t;          // after the wave's last tile: its output partial, [G][D]

  if constexpr (KG::MC) {
    w.sp = a.xs + xs_at(a, bl, kvh * G, 0);
    w.sp_stride = a.xs_stride;
    f32x4 om[1][D / 16];
    float mr[1] = {-INFINITY}, lr[1] = {0.f};
#pragma unroll
    for (int db = 0; db < D / 16; ++db) om[0][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (u < nwf) attn_wave_mfma<D, KT, KG::MF, 1, LOG_CALL>(a, w, bl, 0, kvh, lane, u, nwf, nF, nF, f_loc + (size_t)b * a.Nmax, xsb * TB, om, mr, lr);
    else if (a.t2fmt == 0) attn_wave_mfma<D, KT, Q_INT8, 1, LOG_CALL>(a, w, bl, 0, kvh, lane, u - nwf, nwq, nQ, nQ, a.q_loc + (size_t)b * a.Nmax, colq, om, mr, lr);
    else attn_wave_mfma<D, KT, Q_INT4, 1, LOG_CALL>(a, w, bl, 0, kvh, lane, u - nwf, nwq, nQ, nQ, a.q_loc + (size_t)b * a.Nmax, colq, om, mr, lr);
    park_one<D, G>(om[0], mr[0], lr[0], lane, my_o, sm_ml + wave * 16);
    if (!finite_one<D>(om[0])) {
      if (u < nwf) outputs_plain<D, G, KT, KG::MF, LOG_CALL>(a, w, bl, kvh, lane, u, nwf, nF, f_loc + (size_t)b * a.Nmax, xsb * TB, mr[0], my_o);
      else if (a.t2fmt == 0) outputs_plain<D, G, KT, Q_INT8, LOG_CALL>(a, w, bl, kvh, lane, u - nwf, nwq, nQ, a.q_loc + (size_t)b * a.Nmax, colq, mr[0], my_o);
      else outputs_plain<D, G, KT, Q_INT4, LOG_CALL>(a, w, bl, kvh, lane, u - nwf, nwq, nQ, a.q_loc + (size_t)b * a.Nmax, colq, mr[0], my_o);
    }
  } else {
    float o[G][EV], m_run[G], l_lane[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m_run[h] = -INFINITY; l_lane[h] = 0.f;
#pragma unroll
      for (int e = 0; e < EV; ++e) o[h][e] = 0.f;
    }
    bool o_written = false;
    if (u < nwf) {
      attn_wave<D, G, KG::MF, KT, TR>(a, w, bl, jq, kvh, lane, u, nwf, nF, f_loc + (size_t)b * a.Nmax, xsb * TB, o, m_run, l_lane);
    } else {
      if constexpr (EV == 8) {
        if (a.t2fmt == 0) attn_wave<D, G, Q_INT8, KT, TR>(a, w, bl, jq, kvh, lane, u - nwf, nwq, nQ, a.q_loc + (size_t)b * a.Nmax, colq, o, m_run, l_lane);
        else attn_wave<D, G, Q_INT4, KT, TR>(a, w, bl, jq, kvh, lane, u - nwf, nwq, nQ, a.q_loc + (size_t)b * a.Nmax, colq, o, m_run, l_lane);
      } else {
        // binary32 rows use 4 elements per lane, code rows 8: separate accumulators, parked directly
        float o8[G][8];
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
          for (int e = 0; e < 8; ++e) o8[h][e] = 0.f;
        if (a.t2fmt == 0) attn_wave<D, G, Q_INT8, KT, TR>(a, w, bl, jq, kvh, lane, u - nwf, nwq, nQ, a.q_loc + (size_t)b * a.Nmax, colq, o8, m_run, l_lane);
        else attn_wave<D, G, Q_INT4, KT, TR>(a, w, bl, jq, kvh, lane, u - nwf, nwq, nQ, a.q_loc + (size_t)b * a.Nmax, colq, o8, m_run, l_lane);
        park_rows<D, G, 8, D / 8>(o8, lane, my_o);
        o_written = true;
      }
    }
    // ---- wave partial: sum the row groups and the per-lane denominators, then merge the waves through LDS
    if (!o_written) park_rows<D, G, EV, LPRV>(o, lane, my_o);
    park_stats<G>(m_run, l_lane, lane, sm_ml + wave * 16);
  }
  __syncthreads();
  const int bq = bl * a.n_q + jq;
  float* po = a.part_o + ((size_t)((bq * a.Hkv + kvh) * a.S_total + a.s0 + s) * G) * D;
  for (int i = t; i < G * D; i += NW * 64) {
    const int h = i / D;
    float mb = sm_ml[h];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 16 + h]);
    float acc = 0.f;
    if (mb > -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) {
        const float* src = (const float*)(sm_t + ww * TILE_BYTES) + i;
        acc = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 16 + h] - mb) * LOG2E), src[0], acc);
      }
    }
    po[i] = acc;
  }
  if (t < G) {
    float mb = sm_ml[t];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 16 + t]);
    float ll = 0.f;
    if (mb > -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) ll = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 16 + t] - mb) * LOG2E), sm_ml[ww * 16 + 8 + t], ll);
    }
    float* pm = a.part_ml + ((size_t)((bq * a.Hkv + kvh) * a.S_total + a.s0 + s) * 2) * G;
    pm[t] = mb;
    pm[G + t] = ll;
  }
}

// ---- a whole decode step: one workgroup per (layer, sequence, kv head) pair ----------------------------------------
// With the pairs of all layers of a step in one launch there are enough of them to fill the chip without splitting any,
// and a workgroup that has walked a pair's lists to their end knows the final softmax statistics of its heads.  So it
// writes its output itself, and of the logits, which stay in the LDS, one float per row: the row's weights summed over
// the group's heads.  That is what this kernel is for: written logits (G floats per row, 4-6 % of the bytes) cost far more
// than their bytes beside the row stream (1.6 GB of rows stream in 233 us alone, in 284 us with 25 MB of stores beside them and
// 316 us with 101 MB, in 257 us if all of those come at once at the end).
// The rows' arithmetic runs on the matrix cores, with the G heads as columns of which 16 - G are padding: G dot products and
// G scaled additions per row on the vector ALUs kept these busy for 76 % of the time at seven heads.  us a step with vector /
// matrix instructions, 28 layers, 28/4 heads: 8 x 600 tokens 82 / 68, 5 x 2000 119 / 109, 1 x 1422 33.3 / 30.0; 12 layers, 64/8,
// 1 x 3000 48.9 / 45.0; ten layers, 10/2, 10 x 1500 37.3 / 35.6; 27 layers, 8/8 at head_dim 64, 6 x 1200 88.2 / 87.2.  What the
// stream of rows bounds (14B shape, 48 layers, batch 8, 4112 tokens: 960-1140 us, 6.0 TB/s) is within 1 %.
// Precision: weights enter the product as exact sums of three 16-bit terms, a tile's 32 entries are summed by themselves and
// added to the running output once, quarters of a row's elements are summed by themselves, logits stay unscaled until the
// distance to the maximum is taken, and the exponent's product keeps its remainder.  Outputs against 64 bits, vector / matrix
// instructions, relative 2-norm: 28/4 heads, 8 x 2081, 10 % int8 2.9e-7 / 2.4e-7; 40/8, 8 x 4096, 15 % int8 3.2e-7 / 2.5e-7; 16/4, 1 x
// 16000 4.9e-7 / 2.9e-7; binary16, 40/8, 1 x 8000, int4 4.2e-7 / 2.9e-7; 8/8 at head_dim 64, 2 x 3000 2.45e-7 / 2.25e-7; 10/2, 4 x 700
// 2.4e-7 / 2.1e-7.
// The LDS holds eight 8 KB tile buffers (32 rows of 256 bytes; 64 KB in flight per compute unit stream as fast as 128 KB)
// and the logits of LCAP entries; a longer list parks the rest in memory and reads it back.  The eight waves are divided
// between the lists as in the split launch.
// The pairs that fill the last round of the chip only in part, those of the (layer, sequence) rows from a.whole_rows on, are
// cut into a.S parts of eight waves each (the host's rule: step_tail): a part writes its logits and a partial, as in the
// split launch.
template <int D, int G, bool VEC = false>
struct StepGeo {
  static constexpr int NW = 8, RB = 2 * D, TR = 8192 / RB < 64 ? 8192 / RB : 64, TILE = TR * RB;
  static constexpr int SC = (D / 64) * TR * 4, LT = 2 * TR * 4, P = VEC ? TR * GPad<G>::v * 4 : 0;   // per wave: K or V scales, slot lists, weights
  static constexpr int LDS = 163840, FIXED = NW * (TILE + P + 2 * SC + LT) + NW * 16 * 4 + 8 * 8 + 256;
  static constexpr int LCAP = (LDS - FIXED) / 4 / G / TR * TR;
};
// Caches whose single calls are whole-pair launches (a pair and more for every compute unit): where lists are short a wave has one
// tile or two, and what a tile takes from its arrival on counts for each round of pairs.  With one or two heads a group the vector
// ALUs have a 64-row tile done in half of the time that the matrix cores' wave spends on 16 columns, and keep these caches at head_dim
// 64 up to 1024 tokens.  us a call, matrix / vector instructions: 64 sequences, 8/8 heads, 100 tokens 14.9 / 13.1, 300 19.0 / 16.5,
// 500 20.9 / 19.4, 700 23.8 / 22.7, 1500 40.6 / 42.2, 4000 98 / 105; 4/4, 1000 18.8 / 18.5; 8/4, 300 13.2 / 12.7, 500 14.5 / 14.1; 12/4
// (three a group), 500 14.7 / 14.5; 130 x 300, 4/2 18.4 / 17.3.  Outputs against 64 bits there: 2.0e-7 either way.  At head_dim 128 (64 x
// 300, 4/4 14.1 / 13.7) the matrix cores' are closer, 2.3e-7 / 2.7e-7.
constexpr int VECTOR_TOKENS = 1024;
constexpr bool step_on_vector(int D, int G, int max_tokens) { return D == 64 && G <= 2 && max_tokens <= VECTOR_TOKENS; }
template <int D, int G, int KT, bool VEC>
__global__ __launch_bounds__(512, 2) void k_attn_step(const AttnArgs a) {
  using SG = StepGeo<D, G, VEC>;
  constexpr Mode MF = KT == KT_BF16 ? F_BF16 : F_F16;
  constexpr int NW = SG::NW, TR = SG::TR, TILE = SG::TILE, LCAP = SG::LCAP, EV = Geo<D, MF, TR>::EV;
  static_assert(G * D * 4 <= TILE, "a wave's output partial is parked in its tile buffer");
  __shared__ __attribute__((aligned(16))) char sm_t[NW * TILE];
  __shared__ __attribute__((aligned(16))) char sm_sc[NW * 2 * SG::SC];
  __shared__ __attribute__((aligned(16))) char sm_lt[NW * SG::LT];
  __shared__ __attribute__((aligned(16))) float sm_lg[G * LCAP];
  __shared__ float sm_ml[NW * 16];
  __shared__ float2 sm_fin[8];
  __shared__ __attribute__((aligned(16))) char sm_p[VEC ? NW * SG::P : 16];
  const int kvh = blockIdx.x;
  int bl = blockIdx.y, part = 0;
  // What stands between a workgroup and its first request, all of the arguments asked for at once: they come over the host link,
  // and as the compiler places them, behind the conditions below, one waits for another (64 x 700 tokens, 8/8 heads at head_dim
  // 64, two rounds of pairs: 25.2 us a call so, 23.5 now; 64 x 300, 4/4 at 128, one round: 14.8, 14.1).  A single call's sequence
  // is blockIdx.y; its list lengths are asked for with the rest and corrected in other launches.
  int nl = a.nl, whole_rows = a.whole_rows, S = a.S, B = a.B, Hkv = a.Hkv, Nmax = a.Nmax, t2fmt = a.t2fmt, xs_stride = a.xs_stride;
  int nF = a.nF[bl & (ATTN_ARG_SEQS - 1)], nQ = a.nQ[bl & (ATTN_ARG_SEQS - 1)], nwq = a.nWq[bl & (ATTN_ARG_SEQS - 1)];
  const int *f_new = a.f_loc, *f_old = a.f_loc_old, *q_list = a.q_loc;
  uint64_t old_mask = a.old_mask;
  float* spill = a.xs;
  asm volatile("" : : "s"(nl), "s"(whole_rows), "s"(S), "s"(B), "s"(Hkv), "s"(Nmax), "s"(t2fmt), "s"(xs_stride), "s"(nF), "s"(nQ),
                    "s"(nwq), "s"(f_new), "s"(f_old), "s"(q_list), "s"(old_mask), "s"(spill));
  const bool split = bl >= whole_rows;
  if (split) { const int x = bl - whole_rows; bl = whole_rows + x / S; part = x - (bl - whole_rows) * S; }
  const int li = nl > 1 ? bl / B : 0, b = bl - li * B, pair = bl * Hkv + kvh;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int* f_loc = (((old_mask >> li) & 1) ? f_old : f_new) + (size_t)b * Nmax;
  const int nwv = split ? NW * S : NW, u = part * NW + wave;         // the pair's waves, and which of them this is
  if (B > ATTN_ARG_SEQS) {
    nF = a.cnt[b * CNT_N + C_NF]; nQ = a.cnt[b * CNT_N + C_NQ];
    const int nft = (nF + TR - 1) / TR, nqt = (nQ + TR - 1) / TR;
    nwq = split ? q_waves(nwv, nft, nqt) : q_waves(NW, nft, nqt);   // (a constant number of waves: no division, of 16)
  } else {
    if (nl > 1 || split) { nF = a.nF[b]; nQ = a.nQ[b]; nwq = a.nWq[b]; }
    nwq = split ? nwq >> 16 : nwq & 0xffff;
  }
  const int nft = (nF + TR - 1) / TR, colq = nft * TR;

  WaveLds w;
  w.t = sm_t + wave * TILE; w.p = sm_p + wave * SG::P; w.pa = lds_addr(w.p);
  w.sk = sm_sc + wave * 2 * SG::SC; w.sv = w.sk + SG::SC; w.lt = sm_lt + wave * SG::LT;
  w.ta = lds_addr(w.t); w.ska = lds_addr(w.sk); w.sva = lds_addr(w.sv); w.lta = lds_addr(w.lt);
  w.lga = lds_addr(sm_lg); w.lcap = LCAP;
  w.lim = split ? 0 : LCAP;
  w.sp = split ? a.xt + (size_t)(pair + a.tail0) * G * a.sc_stride : spill + (size_t)pair * G * xs_stride - LCAP;
  w.sp_stride = split ? a.sc_stride : xs_stride;
  float* my_o = (float*)w.t;

  const int nwf = nwv - nwq;
  const int* q_loc = q_list + (size_t)b * Nmax;
  if constexpr (VEC) {
    static_assert(SG::LCAP >= VECTOR_TOKENS + 2 * TB && EV == 8, "all logits in the LDS");
    float o[G][EV], m_run[G], l_lane[G];
#pragma unroll
    for (int h = 0; h < G; ++h) {
      m_run[h] = -INFINITY; l_lane[h] = 0.f;
#pragma unroll
      for (int e = 0; e < EV; ++e) o[h][e] = 0.f;
    }
    if (u < nwf) attn_wave<D, G, MF, KT, TR, true>(a, w, bl, 0, kvh, lane, u, nwf, nF, f_loc, 0, o, m_run, l_lane);
    else if (t2fmt == 0) attn_wave<D, G, Q_INT8, KT, TR, true>(a, w, bl, 0, kvh, lane, u - nwf, nwq, nQ, q_loc, colq, o, m_run, l_lane);
    else attn_wave<D, G, Q_INT4, KT, TR, true>(a, w, bl, 0, kvh, lane, u - nwf, nwq, nQ, q_loc, colq, o, m_run, l_lane);
    park_rows<D, G, EV, Geo<D, MF, TR>::LPRV>(o, lane, my_o);
    park_stats<G>(m_run, l_lane, lane, sm_ml + wave * 16);
  } else {
    f32x4 om[1][D / 16];
    float mr[1] = {-INFINITY}, lr[1] = {0.f};
#pragma unroll
    for (int db = 0; db < D / 16; ++db) om[0][db] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (u < nwf) attn_wave_mfma<D, KT, MF, 1, LOG_STEP>(a, w, bl, 0, kvh, lane, u, nwf, nF, nF, f_loc, 0, om, mr, lr);
    else if (t2fmt == 0) attn_wave_mfma<D, KT, Q_INT8, 1, LOG_STEP>(a, w, bl, 0, kvh, lane, u - nwf, nwq, nQ, nQ, q_loc, colq, om, mr, lr);
    else attn_wave_mfma<D, KT, Q_INT4, 1, LOG_STEP>(a, w, bl, 0, kvh, lane, u - nwf, nwq, nQ, nQ, q_loc, colq, om, mr, lr);
    park_one<D, G>(om[0], mr[0], lr[0], lane, my_o, sm_ml + wave * 16);
    if (!finite_one<D>(om[0])) {
      if (u < nwf) outputs_plain<D, G, KT, MF, LOG_STEP>(a, w, bl, kvh, lane, u, nwf, nF, f_loc, 0, mr[0], my_o);
      else if (t2fmt == 0) outputs_plain<D, G, KT, Q_INT8, LOG_STEP>(a, w, bl, kvh, lane, u - nwf, nwq, nQ, q_loc, colq, mr[0], my_o);
      else outputs_plain<D, G, KT, Q_INT4, LOG_STEP>(a, w, bl, kvh, lane, u - nwf, nwq, nQ, q_loc, colq, mr[0], my_o);
    }
  }
  // ---- merge the waves
  __syncthreads();
  if (split) {
    // a part of a pair: its partial; k_step_scores_parts has the rest of the way
    const size_t sp = (size_t)(pair + a.tail0) * S + part;
    for (int i = t; i < G * D; i += NW * 64) {
      const int h = i / D;
      float mb = sm_ml[h], acc = 0.f;
#pragma unroll
      for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 16 + h]);
      if (mb > -INFINITY) {
#pragma unroll
        for (int ww = 0; ww < NW; ++ww)
          acc = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 16 + h] - mb) * LOG2E), ((const float*)(sm_t + ww * TILE))[i], acc);
      }
      a.part_o[sp * G * D + i] = acc;
    }
    if (t < G) {
      float mb = sm_ml[t], ll = 0.f;
#pragma unroll
      for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 16 + t]);
      if (mb > -INFINITY) {
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) ll = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 16 + t] - mb) * LOG2E), sm_ml[ww * 16 + 8 + t], ll);
      }
      a.part_ml[sp * 2 * G + t] = mb;
      a.part_ml[sp * 2 * G + G + t] = ll;
    }
    return;
  }
  if (t < G) {
    float mb = sm_ml[t], ll = 0.f;
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 16 + t]);
    if (mb > -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) ll = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 16 + t] - mb) * LOG2E), sm_ml[ww * 16 + 8 + t], ll);
    }
    // no live position at all (a forced plan): zeros, not 0/0
    sm_fin[t] = make_float2(mb > -INFINITY ? mb : 0.f, ll > 0.f ? 1.0f / ll : 0.f);
  }
  __syncthreads();
  for (int i = t; i < G * D; i += NW * 64) {
    const int h = i / D;
    const float2 fin = sm_fin[h];
    float acc = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) {
      const float* src = (const float*)(sm_t + ww * TILE) + i;
      acc = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 16 + h] - fin.x) * LOG2E), src[0], acc);
    }
    acc *= fin.y;
    const size_t oi = ((size_t)bl * a.o_bs + kvh * G) * D + i;
    if (a.out_kind == KT_BF16) ((uint16_t*)a.out)[oi] = f32_to_bf16(acc);
    else if (a.out_kind == KT_F16) ((_Float16*)a.out)[oi] = (_Float16)acc;    // round to nearest even
    else ((float*)a.out)[oi] = acc;
  }
  // ---- the rows' weights, summed over the group's heads
  const float pen = a.red ? a.red_w * (float)G / (float)(nF + nQ) : 0.f;
  float2 fin[G];
#pragma unroll
  for (int h = 0; h < G; ++h) fin[h] = sm_fin[h];
  const size_t pr = (size_t)bl * a.Hkv + kvh;
  for (int c = t; c < colq + nQ; c += NW * 64) {
    if (c >= nF && c < colq) continue;
    float x[G], s = 0.f;
    if (c < LCAP) {
#pragma unroll
      for (int h = 0; h < G; ++h) x[h] = sm_lg[h * LCAP + c];
    } else {
#pragma unroll
      for (int h = 0; h < G; ++h) x[h] = a.xs[(pr * G + h) * a.xs_stride + (c - LCAP)];
    }
#pragma unroll
    for (int h = 0; h < G; ++h) s += exp_le0(fmaf(x[h], a.softmax_scale, -fin[h].x)) * fin[h].y;
    if (a.vnorm || a.red) {
      const int pos = c < nF ? a.f_pos[(size_t)b * a.Nmax + c] : a.q_pos[(size_t)b * a.Nmax + (c - colq)];
      if (a.vnorm) s *= a.vnorm[pr * a.Nmax + pos];         // value-aware scorer: times the norm of the value row the group reads
      if (a.red) s = fmaf(-pen, a.red[pr * a.Nmax + pos], s);   // redundancy-penalised: each head takes red_w * rho / (positions attended) off
    }
    a.sc[pr * a.sc_stride + c] = s;
  }
}

// ---- a chunk of query tokens, 16-bit rows: every wave on the matrix cores -------------------------------------------
// The chunk's a.cq * a.G columns go in groups of 16 * NCB along grid z (x batch), whatever token a group begins with, so
// that one launch serves them all: 13 tokens of seven heads are three groups of 32 columns.  Eight waves per workgroup, two
// per SIMD, with 8 KB tiles.  A wave's result arrives complete (no row-group partials): [column][D], parked in the LDS.
// LOG: one group of columns; the logits go to memory and attn_finish_chunk reads them.  Else no logits leave the kernel: a
// float per row and column is a quarter of the rows' bytes at 32 columns and costs more than that (stores beside the row
// stream), while the score launch below has the products again for half of the rows' bytes, once for all columns.
// Registers with two blocks of columns at head_dim 128: 250-255 of 256 in bfloat16; binary16 spills one (six with LOG).
constexpr int MC_WAVES = 8;
constexpr int mc_tile_rows(int D) { return 8192 / (2 * D); }
constexpr int chunk_blocks(int ncol) { return ncol <= 16 ? 1 : 2; }      // of 16 columns, per workgroup
// With one group of columns the logits are written (LOG), with more they are not.  us a call, written / not: 8 sequences x 16384
// tokens, 12/2 heads, two query tokens (12 columns) 41 / 61; 32 x 1000, 8/8, two (2) 30 / 45; 8 x 4133, 40/8, four (20) 44 / 47.
// From two groups on: 8 x 2081, 28/4, 13 (91 columns) 105 written (a launch pair per group) / 39; over 172 shapes 1.1 to 4.5
// times as fast, least with 48 columns.  (attn_finish_chunk takes 16 tokens at most.)
constexpr bool chunk_logits(int cq, int G) { return cq * G <= 32 && cq <= 16; }
template <int D, int KT, int NCB, bool LOG>
__global__ __launch_bounds__(MC_WAVES * 64, MC_WAVES / 4) void k_attn_tiered_mc(const AttnArgs a) {
  constexpr int NW = MC_WAVES, TR = mc_tile_rows(D), TILE = 8192, SC = (D / 64) * TR * 4;
  constexpr int PART = 16 * NCB * D * 4, TILE_BYTES = PART > TILE ? PART : TILE;   // a wave's output partial takes its tile buffer's place
  constexpr Mode MF = KT == KT_BF16 ? F_BF16 : F_F16;
  __shared__ __attribute__((aligned(16))) char sm_t[NW * TILE_BYTES];
  __shared__ __attribute__((aligned(16))) char sm_sc[NW * 2 * SC];
  __shared__ __attribute__((aligned(16))) char sm_lt[NW * 2 * TR * 4];
  __shared__ float sm_ml[NW * 64];                       // per wave: m of 32 columns, then l
  const int s = blockIdx.x, kvh = blockIdx.y;
  const int b = a.groups > 1 ? (int)blockIdx.z / a.groups : (int)blockIdx.z, jz = a.groups > 1 ? (int)blockIdx.z % a.groups : 0;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int nF, nQ;
  if (a.B <= ATTN_ARG_SEQS) { nF = a.nF[b]; nQ = a.nQ[b]; }
  else { nF = a.cnt[b * CNT_N + C_NF] - a.trim; nQ = a.cnt[b * CNT_N + C_NQ]; }
  // this group's columns; its last one's token is cq - 1 - token positions older than the launch's last, and that many
  // entries at the end of list F are not the group's to see (its earlier tokens cut off more, column by column)
  const int ncol = a.cq * a.G, c0 = jz * 16 * NCB, nc = ncol - c0 < 16 * NCB ? ncol - c0 : 16 * NCB;
  const int nFw = nF - (a.cq - 1 - (c0 + nc - 1) / a.G);
  const int nwv = a.S * NW;
  const int nwq = a.B <= ATTN_ARG_SEQS ? a.nWq[b] : q_waves(nwv, (nF + TR - 1) / TR, (nQ + TR - 1) / TR), nwf = nwv - nwq;
  const int u = s * NW + wave;

  WaveLds w;
  w.t = sm_t + wave * TILE_BYTES;
  w.sk = sm_sc + wave * 2 * SC; w.sv = w.sk + SC; w.lt = sm_lt + wave * 2 * TR * 4;
  w.ta = lds_addr(w.t); w.ska = lds_addr(w.sk); w.sva = lds_addr(w.sv); w.lta = lds_addr(w.lt);
  w.p = nullptr; w.pa = 0;
  float* my_o = (float*)w.t;          // after the wave's last tile: its output partial, [column][D]

  f32x4 om[NCB][D / 16];
  float mr[NCB], lr[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    mr[cb] = -INFINITY; lr[cb] = 0.f;
#pragma unroll
    for (int db = 0; db < D / 16; ++db) om[cb][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  if (u < nwf) attn_wave_mfma<D, KT, MF, NCB, LOG ? LOG_XS : LOG_NONE>(a, w, b, c0, kvh, lane, u, nwf, nF, nFw, (a.old_mask ? a.f_loc_old : a.f_loc) + (size_t)b * a.Nmax, 0, om, mr, lr);
  else if (a.t2fmt == 0) attn_wave_mfma<D, KT, Q_INT8, NCB, LOG ? LOG_XS : LOG_NONE>(a, w, b, c0, kvh, lane, u - nwf, nwq, nQ, nQ, a.q_loc + (size_t)b * a.Nmax, ((nF + 63) >> 6) * TB, om, mr, lr);
  else attn_wave_mfma<D, KT, Q_INT4, NCB, LOG ? LOG_XS : LOG_NONE>(a, w, b, c0, kvh, lane, u - nwf, nwq, nQ, nQ, a.q_loc + (size_t)b * a.Nmax, ((nF + 63) >> 6) * TB, om, mr, lr);
  // ---- wave partial into LDS: lane (n, kb) has the statistics of column 16*cb + n and the outputs of columns
  // 16*cb + 4*kb + j, element 16*db + n
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) {
    const float ls = quad_sum(lr[cb]);
    const int col = 16 * cb + lane;
    if (lane < 16 && col < nc) { sm_ml[wave * 64 + col] = mr[cb]; sm_ml[wave * 64 + 32 + col] = ls; }
#pragma unroll
    for (int db = 0; db < D / 16; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int c = 16 * cb + 4 * (lane >> 4) + j;
        if (c < nc) my_o[c * D + 16 * db + (lane & 15)] = om[cb][db][j];
      }
  }
  __syncthreads();
  // ---- merge the waves: one split partial (m, l, o[D]) per column; LOG: laid out by query token, as attn_finish_chunk merges them
  const size_t sp = (size_t)(b * a.Hkv + kvh) * a.S + s;
  const float inv_g = 1.0f / (float)a.G;
  const auto by_token = [&](int jq) { return ((size_t)(b * a.cq + jq) * a.Hkv + kvh) * a.S + s; };
  for (int i = t; i < nc * D; i += NW * 64) {
    const int col = i / D;
    float mb = sm_ml[col];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 64 + col]);
    float acc = 0.f;
    if (mb > -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww)
        acc = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 64 + col] - mb) * LOG2E), ((const float*)(sm_t + ww * TILE_BYTES))[i], acc);
    }
    if constexpr (LOG) { const int jq = small_div(col, inv_g); a.part_o[(by_token(jq) * a.G + (col - jq * a.G)) * D + i % D] = acc; }
    else a.part_o[(sp * ncol + c0) * D + i] = acc;
  }
  if (t < nc) {
    float mb = sm_ml[t];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) mb = fmaxf(mb, sm_ml[ww * 64 + t]);
    float ll = 0.f;
    if (mb > -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < NW; ++ww) ll = fmaf(__builtin_amdgcn_exp2f((sm_ml[ww * 64 + t] - mb) * LOG2E), sm_ml[ww * 64 + 32 + t], ll);
    }
    const int jq = small_div(t, inv_g);
    float* pm = LOG ? a.part_ml + by_token(jq) * 2 * a.G + (t - jq * a.G) : a.part_ml + sp * 2 * ncol + c0 + t;
    pm[0] = mb;
    pm[LOG ? a.G : ncol] = ll;
  }
}

// ---- the scores of a chunk (16-bit rows), and its outputs ------------------------------------------------------------
// Grid (runs of tpw tiles of list F, then of list Q, of CS_ROWS entries, then output workgroups; B).  A workgroup has its K rows once more, for all
// kv heads and all of the chunk's columns, and adds every entry's weights, summed, to its score: wave w takes kv heads
// w / nsub, + 8 / nsub, ... and of their columns blocks w % nsub, + nsub, ...; a kv head's blocks, then the kv heads are
// added in that order.  The weights are exp2 of the same products (same instructions, same operand order) less the merged
// maximum, times the merged 1 / l: those that went into the output but for one rounding of the scaled logit, which the fma
// that takes the maximum off does not make.  The last workgroups of a
// sequence (n_out) merge its splits into out; beside the rows, in the other workgroups, that took 4 us more.
// Bound by rows arriving, half of what the launch before fetched.  Two tiles per wave are in flight (64-128 KB per compute
// unit); nothing else goes through the vector memory pipe in the loop, because waiting for it would mean waiting for the
// rows before it: the query vectors stay in registers, CS_QB blocks at a time, slots and statistics come from the LDS.
constexpr int CHUNK_TOKENS = 32;                   // query tokens of a launch, at most
constexpr int CS_THREADS = 512, CS_WAVES = CS_THREADS / 64;
constexpr int CS_RB = 2, CS_ROWS = 16 * CS_RB, CS_QB = 4;
constexpr size_t cs_tiles(int D) { return CS_WAVES * 2 * CS_ROWS * 2 * D; }   // bytes of the tile buffers
constexpr size_t cs_lds(int D) { return 163840 - cs_tiles(D); }               // what is left beside them
// (m, 1/l) of one column out of ns split partials `stride` floats apart (l follows m by `lofs`), by one wave: all lanes get them
__device__ __forceinline__ void merge_stats_wave(const float* __restrict__ src, int ns, size_t stride, int lofs, int lane, float& m, float& il) {
  float mx[1] = {-INFINITY}, lsum = 0.f;
  for (int k = lane; k < ns; k += 64) mx[0] = fmaxf(mx[0], src[k * stride]);
  wave_max_all<1>(mx);
  const float mm = rdlane(mx[0], 63);
  if (mm > -INFINITY)
    for (int k = lane; k < ns; k += 64) lsum = fmaf(src[k * stride + lofs], __builtin_amdgcn_exp2f((src[k * stride] - mm) * LOG2E), lsum);
  lsum = wave_sum(lsum);
  m = mm > -INFINITY ? mm : 0.f;
  il = lsum > 0.f ? 1.0f / lsum : 0.f;
}
// the same by one thread
__device__ __forceinline__ void merge_stats_thread(const float* __restrict__ src, int ns, size_t stride, int lofs, float& m, float& il) {
  float mm = -INFINITY, ll = 0.f;
  if (ns <= 4) {
    float mv[4], lv[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) { mv[k] = k < ns ? src[k * stride] : -INFINITY; lv[k] = k < ns ? src[k * stride + lofs] : 0.f; }
    mm = fmaxf(fmaxf(mv[0], mv[1]), fmaxf(mv[2], mv[3]));
    if (mm > -INFINITY) {
#pragma unroll
      for (int k = 0; k < 4; ++k) ll = fmaf(lv[k], __builtin_amdgcn_exp2f((mv[k] - mm) * LOG2E), ll);
    }
  } else {
#pragma unroll 8
    for (int k = 0; k < ns; ++k) mm = fmaxf(mm, src[k * stride]);
    if (mm > -INFINITY) {
#pragma unroll 8
      for (int k = 0; k < ns; ++k) ll = fmaf(src[k * stride + lofs], __builtin_amdgcn_exp2f((src[k * stride] - mm) * LOG2E), ll);
    }
  }
  m = mm > -INFINITY ? mm : 0.f;
  il = ll > 0.f ? 1.0f / ll : 0.f;
}
// waves that share a kv head's columns
__host__ __device__ inline int chunk_nsub(int Hkv, int ncol) {
  const int blocks = (ncol + 15) / 16, n = Hkv >= CS_WAVES ? 1 : CS_WAVES / Hkv;
  return n < blocks ? n : blocks;
}
inline size_t chunk_scores_lds(int Hq, int Hkv, int cq, int G, int tpw) {
  return (size_t)(cq * Hq + 1) / 2 * 16 + ((size_t)Hkv * chunk_nsub(Hkv, cq * G) + 1) * tpw * CS_ROWS * 4 + CS_WAVES * 4 * CS_ROWS * 4;
}
// the workgroup's share (of n_wgs, number u) of the output rows (kv head, column) of sequence b
template <int D>
__device__ __forceinline__ void chunk_outputs(const AttnArgs& a, int b, int u, int n_wgs, float* sm_red) {
  constexpr int PAR = CS_THREADS / D;                                        // rows, or shares of one row's splits, side by side
  const int t = threadIdx.x, lane = t & 63, d = t % D, g = t / D, ncol = a.cq * a.G, rows = a.Hkv * ncol, S = a.S;
  const int rpw = (rows + n_wgs - 1) / n_wgs, r0 = u * rpw, r1 = r0 + rpw < rows ? r0 + rpw : rows;
  const size_t mls = (size_t)2 * ncol;                                       // floats between a pair's split statistics
  const float inv_g = 1.0f / (float)a.G, inv_c = 1.0f / (float)ncol;
  auto store = [&](int kvh, int col, float v) {
    const int jq = small_div(col, inv_g);
    const size_t oi = ((size_t)b * a.o_bs + (size_t)jq * a.Hq + kvh * a.G + (col - jq * a.G)) * D + d;
    if (a.out_kind == KT_BF16) ((uint16_t*)a.out)[oi] = f32_to_bf16(v);
    else if (a.out_kind == KT_F16) ((_Float16*)a.out)[oi] = (_Float16)v;
    else ((float*)a.out)[oi] = v;
  };
  if (S <= 4) {
    constexpr int NRW = 4;                                                   // rows of a thread whose loads are in flight together
    for (int rr = r0 + g; rr < r1; rr += NRW * PAR) {
      int kvh[NRW], col[NRW];
      float po[NRW][4], mv[NRW][4], lv[NRW][4];
#pragma unroll
      for (int i = 0; i < NRW; ++i) {
        const int r = rr + i * PAR < r1 ? rr + i * PAR : r0;
        kvh[i] = small_div(r, inv_c); col[i] = r - kvh[i] * ncol;
        const size_t sp = ((size_t)b * a.Hkv + kvh[i]) * S;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          const float* ml = a.part_ml + (sp + (k < S ? k : 0)) * mls + col[i];
          po[i][k] = a.part_o[((sp + (k < S ? k : 0)) * ncol + col[i]) * D + d];
          mv[i][k] = k < S ? ml[0] : -INFINITY; lv[i][k] = k < S ? ml[ncol] : 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < NRW; ++i) {
        if (rr + i * PAR >= r1) break;
        const float mm = fmaxf(fmaxf(mv[i][0], mv[i][1]), fmaxf(mv[i][2], mv[i][3]));
        float ll = 0.f, acc = 0.f;
        if (mm > -INFINITY) {
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const float w = __builtin_amdgcn_exp2f((mv[i][k] - mm) * LOG2E);
            ll = fmaf(lv[i][k], w, ll); acc = fmaf(w, po[i][k], acc);
          }
        }
        store(kvh[i], col[i], ll > 0.f ? acc * (1.0f / ll) : 0.f);
      }
    }
  } else {
    for (int r = r0; r < r1; ++r) {
      const int kvh = small_div(r, inv_c), col = r - kvh * ncol;
      const size_t sp = ((size_t)b * a.Hkv + kvh) * S;
      float m, il, acc = 0.f;
      merge_stats_wave(a.part_ml + sp * mls + col, S, mls, ncol, lane, m, il);
#pragma unroll 4
      for (int k = g; k < S; k += PAR) acc = fmaf(__builtin_amdgcn_exp2f((a.part_ml[(sp + k) * mls + col] - m) * LOG2E), a.part_o[((sp + k) * ncol + col) * D + d], acc);
      sm_red[t] = acc;
      __syncthreads();
      if (g == 0) {
        float tot = acc;
#pragma unroll
        for (int k = 1; k < PAR; ++k) tot += sm_red[k * D + d];
        store(kvh, col, tot * il);
      }
      __syncthreads();
    }
  }
}

// Entries e0 .. of one list, tpw tiles, by the whole workgroup.
template <int D, int KT, Mode M>
__device__ __forceinline__ void chunk_scores(const AttnArgs& a, int b, int e0, int tpw, int nF, int nQ, char* sm_t, char* sm) {
  constexpr bool IS_Q = (M == Q_INT8 || M == Q_INT4);
  constexpr int RB = 2 * D, NKS = D / 32, CRB = !IS_Q ? RB : (M == Q_INT8 ? D : D / 2);
  constexpr int SCD = (M == Q_INT8) ? 1 : (M == Q_INT4) ? D / 64 : 0;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n = lane & 15, kb = lane >> 4, ncol = a.cq * a.G, S = a.S, n_list = IS_Q ? nQ : nF;
  const int prow = tpw * CS_ROWS, n_rows = n_list - e0 < prow ? n_list - e0 : prow, nt = (n_rows + CS_ROWS - 1) / CS_ROWS;
  const int nsub = chunk_nsub(a.Hkv, ncol), kv_step = CS_WAVES / nsub, sub = wave % nsub, kvh0 = wave / nsub;
  const int blocks = (ncol + 15) / 16, my_blocks = (blocks - sub + nsub - 1) / nsub, ng = (my_blocks + CS_QB - 1) / CS_QB;
  const float inv_g = 1.0f / (float)a.G, inv_c = 1.0f / (float)ncol;
  float2* sm_st = (float2*)sm;                                               // (m, 1/l) of every (kv head, column)
  float* sm_part = (float*)(sm_st + ((a.Hkv * ncol + 1) & ~1));               // [kv head][sub][prow]: sums over a block set's columns
  int* sm_list = (int*)(sm_part + a.Hkv * nsub * prow);                      // slots of the workgroup's entries
  char* sm_scl = (char*)(sm_list + prow) + wave * 4 * CS_ROWS * 4;      // a wave's scales, two tiles
  const int* list = (IS_Q ? a.q_loc : a.old_mask ? a.f_loc_old : a.f_loc) + (size_t)b * a.Nmax + e0;

  // The K rows come in by direct-to-LDS loads, 1 KB of consecutive pieces per instruction (the operand's own order, 16 rows
  // at a time, keeps the address path busy four times as long).  F: as in attn_wave_mfma, eight rows x 128 bytes, the pieces
  // rotated.  Code rows: whole rows, the 16-byte pieces rotated by row.
  constexpr int LPR = CRB / 16, RPP = 64 / LPR, NP = CS_ROWS * CRB / 1024, KU = RB / 128, TILE = CS_ROWS * CRB;
  constexpr int NR = IS_Q ? NP : CS_ROWS / 8;                                // rows of a tile that this lane fetches from
  constexpr int ROWP = IS_Q ? RPP : 8;                                       // ... and their distance
  const int row0 = IS_Q ? lane / LPR : lane >> 3, srow = lane & (CS_ROWS - 1);
  char* tb = sm_t + wave * (2 * CS_ROWS * RB);
  uint32_t col16[2];
  if constexpr (IS_Q) {
    col16[0] = col16[1] = (uint32_t)((lane - (M == Q_INT8 ? row0 : row0 >> 1)) & (LPR - 1)) * 16u;   // (RPP is a multiple of the rotation's period)
  } else {
    const int r = lane & 7;
    col16[0] = (uint32_t)((r + 2 * (row0 >> 1)) & 7) * 16u; col16[1] = (uint32_t)((r + 2 * (row0 >> 1) + 1) & 7) * 16u;
  }
  // the tile that is fetched next: tile f_ti of the workgroup's, for kv head f_kvh and the f_g-th set of its blocks
  int f_ti = 0, f_g = 0, f_kvh = kvh0;
  bool f_more = wave < kv_step * nsub && kvh0 < a.Hkv;
  auto fetch = [&](int buf, const int (&slot)[NR], int sslot) {              // slots (none: -1, which gives zeros)
    const size_t pr = (size_t)b * a.Hkv + f_kvh;
    const __amdgpu_buffer_rsrc_t rk = IS_Q ? make_rsrc(a.c2K + pr * a.cap2 * CRB, (uint32_t)a.cap2 * CRB) : make_rsrc(a.fpK + pr * a.capF * RB, (uint32_t)a.capF * RB);
#pragma unroll
    for (int i = 0; i < NP; ++i)
      dma<16>(rk, tb + buf * TILE + i * 1024, (uint32_t)slot[IS_Q ? i : i / KU] * (uint32_t)CRB + (IS_Q ? 0 : (i % KU) * 128) + col16[(i / KU) & 1], 0);
    if constexpr (IS_Q) {
      const __amdgpu_buffer_rsrc_t rs = make_rsrc(a.s2K + pr * a.cap2 * a.sb, (uint32_t)a.cap2 * a.sb);
      if (lane < CS_ROWS) {
#pragma unroll
        for (int j = 0; j < SCD; ++j) dma<4>(rs, sm_scl + (buf * 2 + j) * (CS_ROWS * 4), (uint32_t)sslot * (uint32_t)a.sb + 4 * j, 0);
      }
    }
    if (++f_ti == nt) {
      f_ti = 0;
      if (++f_g == ng) { f_g = 0; f_kvh += kv_step; f_more = f_kvh < a.Hkv; }
    }
  };
  constexpr int NOPS = NP + SCD;                                             // vector-memory operations of a fetch
  // addresses of a lane's operand pieces: row n of a 16-row block, elements 32 * ks + 8 * kb .. + 7
  uint32_t k_rd[NKS];
  {
    const uint32_t ta = lds_addr(tb);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      if constexpr (!IS_Q) { const int ii = n >> 3, gg = n & 7, rot = 2 * (gg >> 1) + ii; k_rd[ks] = ta + (ii * KU + (ks >> 1)) * 1024 + (8 * gg + ((4 * (ks & 1) + kb - rot) & 7)) * 16; }
      else if constexpr (M == Q_INT8) k_rd[ks] = ta + n * CRB + ((2 * ks + (kb >> 1) + n) & (LPR - 1)) * 16 + (kb & 1) * 8;
      else k_rd[ks] = ta + n * CRB + ((ks + (n >> 1)) & (LPR - 1)) * 16 + kb * 4;
    }
  }
  const uint32_t part_a = lds_addr(sm_part), list_a = lds_addr(sm_list), scl_a = lds_addr(sm_scl);
  {
    int s0[NR], s1[NR], z0 = -1, z1 = -1;                                    // the first two fetches: tiles 0 and 1, or 0 again
    const int o1 = nt > 1 ? CS_ROWS : 0;
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int r = row0 + i * ROWP;
      s0[i] = r < n_rows ? list[r] : -1;
      s1[i] = o1 + r < n_rows ? list[o1 + r] : -1;
    }
    if constexpr (IS_Q) { z0 = srow < n_rows ? list[srow] : -1; z1 = o1 + srow < n_rows ? list[o1 + srow] : -1; }
    if (f_more) fetch(0, s0, z0);
    if (f_more) fetch(1, s1, z1);
  }
  int my_slot = -1, pos = 0;                                                 // of entry e0 + t
  if (t < n_rows) { my_slot = list[t]; pos = (IS_Q ? a.q_pos : a.f_pos)[(size_t)b * a.Nmax + e0 + t]; }

  // the statistics of the columns
  const size_t mls = (size_t)2 * ncol;                                       // floats between a pair's split statistics
  const float* ml = a.part_ml + (size_t)b * a.Hkv * S * mls;
  if (S > 16) {
    for (int i = wave; i < a.Hkv * ncol; i += CS_WAVES) {
      const int kvh = i / ncol;
      float m, il;
      merge_stats_wave(ml + (size_t)kvh * S * mls + (i - kvh * ncol), S, mls, ncol, lane, m, il);
      if (lane == 0) sm_st[i] = make_float2(m, il);
    }
  } else {
    for (int i = t; i < a.Hkv * ncol; i += CS_THREADS) {
      const int kvh = small_div(i, inv_c);
      float m, il;
      merge_stats_thread(ml + (size_t)kvh * S * mls + (i - kvh * ncol), S, mls, ncol, m, il);
      sm_st[i] = make_float2(m, il);
    }
  }
  if (t < prow) sm_list[t] = my_slot;
  __syncthreads();
  float score = 0.f;
  if (t < n_rows) score = a.score[(size_t)b * a.Nmax + pos];
  if (wave < kv_step * nsub) {
    int buf = 0;
    for (int kvh = kvh0; kvh < a.Hkv; kvh += kv_step)
      for (int g = 0; g < ng; ++g) {
        u32x4 q[CS_QB][NKS];
        float2 st[CS_QB];
        int seen[CS_QB];                                                     // entries the column's query sees
#pragma unroll
        for (int i = 0; i < CS_QB; ++i) {
          const int blk = sub + (g * CS_QB + i) * nsub, col = blk * 16 + n;
          const u32x4* qp = (const u32x4*)a.xs + ((size_t)(b * a.Hkv + kvh) * blocks + (blk < blocks ? blk : 0)) * (NKS * 64) + lane;
#pragma unroll
          for (int ks = 0; ks < NKS; ++ks) q[i][ks] = qp[ks * 64];
          st[i] = sm_st[kvh * ncol + (col < ncol ? col : ncol - 1)];
          if (col >= ncol) st[i].y = 0.f;                                    // the last column once more, with no weight
          seen[i] = (IS_Q ? n_list : col < ncol ? nF - (a.cq - 1 - small_div(col, inv_g)) : nF) - e0 - 4 * kb;
        }
        for (int ti = 0; ti < nt; ++ti, buf ^= 1) {
          // this tile's rows are in (one later fetch at most has been asked for: the one f_ runs ahead by)
          const bool last = ti + 1 == nt && g + 1 == ng && kvh + kv_step >= a.Hkv;
          if (last) wait_vm<0>(); else wait_vm<NOPS>();
          const uint32_t kofs = (uint32_t)buf * TILE;
          u32x4 k[CS_RB][NKS], ksc[IS_Q ? SCD : 1][CS_RB];
          int slot[NR], sslot = -1;
          const uint32_t la = list_a + (uint32_t)(f_ti * CS_ROWS) * 4u;
          static_for<NR>([&](auto ic) { constexpr int i = decltype(ic)::value; slot[i] = (int)lds_rd32<i * ROWP * 4>(la + row0 * 4u); });
          if constexpr (IS_Q) {
            sslot = (int)lds_rd32<0>(la + srow * 4u);
            static_for<SCD>([&](auto jc) {
              constexpr int j = decltype(jc)::value;
              static_for<CS_RB>([&](auto rc) { constexpr int rb = decltype(rc)::value; ksc[j][rb] = lds_rd128<j * CS_ROWS * 4 + rb * 64>(scl_a + buf * (2 * CS_ROWS * 4) + kb * 16u); });
            });
          }
          u32x2 c8[CS_RB][NKS];
          uint32_t c4[CS_RB][NKS];
          static_for<CS_RB>([&](auto rc) {
            constexpr int rb = decltype(rc)::value;
            static_for<NKS>([&](auto kc) {
              constexpr int ks = decltype(kc)::value;
              if constexpr (!IS_Q) k[rb][ks] = lds_rd128<rb * 2 * KU * 1024>(k_rd[ks] + kofs);
              else if constexpr (M == Q_INT8) c8[rb][ks] = lds_rd64<rb * 16 * CRB>(k_rd[ks] + kofs);
              else c4[rb][ks] = lds_rd32<rb * 16 * CRB>(k_rd[ks] + kofs);
            });
          });
          lds_wait();
#pragma unroll
          for (int i = 0; i < NR; ++i) { uint32_t v = (uint32_t)slot[i]; tie(v); slot[i] = (int)v; }
          if constexpr (IS_Q) {
            uint32_t v = (uint32_t)sslot;
            tie(v);
            sslot = (int)v;
#pragma unroll
            for (int j = 0; j < SCD; ++j) tie(ksc[j]);
          }
#pragma unroll
          for (int rb = 0; rb < CS_RB; ++rb) {
            if constexpr (!IS_Q) tie(k[rb]);
            else if constexpr (M == Q_INT8) tie(c8[rb]);
            else tie(c4[rb]);
          }
          if (f_more) fetch(buf, slot, sslot);                               // the buffer has been read
          if constexpr (IS_Q) {
#pragma unroll
            for (int rb = 0; rb < CS_RB; ++rb)
#pragma unroll
              for (int ks = 0; ks < NKS; ++ks) {
                if constexpr (M == Q_INT8) {
                  uint32_t w0, w1, w2, w3;
                  widen_int8<KT>(c8[rb][ks].x, w0, w1);
                  widen_int8<KT>(c8[rb][ks].y, w2, w3);
                  k[rb][ks] = u32x4{w0, w1, w2, w3};
                } else {
                  k[rb][ks] = widen_int4<KT>(c4[rb][ks]);
                }
              }
          }
          const bool edge = (ti + 1) * CS_ROWS > n_list - (IS_Q ? 0 : a.cq - 1) - e0;   // some column does not see the whole tile
          float acc[CS_RB][4];
#pragma unroll
          for (int rb = 0; rb < CS_RB; ++rb)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[rb][j] = 0.f;
#pragma unroll
          for (int i = 0; i < CS_QB; ++i) {
            if (g * CS_QB + i >= my_blocks) break;
            const int lim = seen[i] - ti * CS_ROWS;
            f32x4 xx[CS_RB];
#pragma unroll
            for (int rb = 0; rb < CS_RB; ++rb) {
              f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
              for (int ks = 0; ks < NKS; ++ks) {
                if constexpr (M == Q_INT4) {
                  const f32x4 part = mfma_16x16x32<KT>(k[rb][ks], q[i][ks], f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
                  for (int j = 0; j < 4; ++j) x[j] = fmaf(half_of(elem(ksc[ks >> 1][rb], j), ks & 1), part[j], x[j]);
                } else {
                  x = mfma_16x16x32<KT>(k[rb][ks], q[i][ks], x);
                }
              }
              xx[rb] = x;
            }
#pragma unroll
            for (int rb = 0; rb < CS_RB; ++rb)
#pragma unroll
              for (int j = 0; j < 4; ++j) {
                float x = xx[rb][j];
                if constexpr (M == Q_INT8) x *= elem_f(ksc[0][rb], j);
                x = fmaf(x, a.softmax_scale, -st[i].x);
                if (edge) x = 16 * rb + j < lim ? x : -INFINITY;
                acc[rb][j] = fmaf(__builtin_amdgcn_exp2f(x * LOG2E), st[i].y, acc[rb][j]);
              }
          }
          // summed over the block's 16 columns: lane (n, kb) of the first eight n keeps entry 16 * (n / 4) + 4 * kb + n % 4
          float v = 0.f;
#pragma unroll
          for (int rb = 0; rb < CS_RB; ++rb)
#pragma unroll
            for (int j = 0; j < 4; ++j) { const float tot = group_sum<16>(acc[rb][j]); v = n == 4 * rb + j ? tot : v; }
          const uint32_t at = part_a + (uint32_t)((kvh * nsub + sub) * prow + ti * CS_ROWS + 16 * (n >> 2) + 4 * kb + (n & 3)) * 4u;
          if (n < 4 * CS_RB) {
            if (g > 0) { uint32_t old = lds_rd32<0>(at); lds_wait(); tie(old); v = __builtin_bit_cast(float, old) + v; }
            lds_wr32(at, __builtin_bit_cast(uint32_t, v));
          }
        }
      }
  }
  lds_wait();
  __syncthreads();
  if (t < n_rows) {
    float pen = 0.f;
    if (a.red)           // redundancy-penalised scorers: every token that sees the entry takes red_w * rho / (positions attended) off per head
      for (int jt = 0; jt < a.cq; ++jt) {
        const int later = a.cq - 1 - jt;
        if (IS_Q || e0 + t < nF - later) pen += a.red_w * (float)a.G / (float)(nF - later + nQ);
      }
    float sum = 0.f;
    for (int kvh = 0; kvh < a.Hkv; ++kvh) {
      const float* src = sm_part + kvh * nsub * prow + t;
      float s = src[0];
      for (int w = 1; w < nsub; ++w) s += src[w * prow];
      const size_t o = ((size_t)b * a.Hkv + kvh) * a.Nmax + pos;
      if (a.vnorm) s *= a.vnorm[o];                // value-aware scorer: times the norm of the value row the heads read
      if (a.red) s = fmaf(-pen, a.red[o], s);
      sum += s;
    }
    a.score[(size_t)b * a.Nmax + pos] = score + a.score_scale * sum;
  }
}

template <int D, int KT>
__global__ __launch_bounds__(CS_THREADS, 2) void k_attn_chunk_scores(const AttnArgs a, int n_wgs, int tpw) {
  extern __shared__ __attribute__((aligned(16))) char sm_cs[];
  __shared__ __attribute__((aligned(16))) char sm_t[cs_tiles(D)];   // K rows of each wave, two tiles
  constexpr Mode MF = KT == KT_BF16 ? F_BF16 : F_F16;
  const int b = blockIdx.y, u = blockIdx.x, rows = tpw * CS_ROWS;
  int nF = a.nF[b & (ATTN_ARG_SEQS - 1)], nQ = a.nQ[b & (ATTN_ARG_SEQS - 1)];
  if (a.B > ATTN_ARG_SEQS) { nF = a.cnt[b * CNT_N + C_NF] - a.trim; nQ = a.cnt[b * CNT_N + C_NQ]; }
  if (u >= n_wgs) { chunk_outputs<D>(a, b, u - n_wgs, gridDim.x - n_wgs, (float*)sm_cs); return; }
  const int wf = (nF + rows - 1) / rows;
  if (u >= wf + (nQ + rows - 1) / rows) return;
  if (u < wf) chunk_scores<D, KT, MF>(a, b, u * rows, tpw, nF, nQ, sm_t, sm_cs);
  else if (a.t2fmt == 0) chunk_scores<D, KT, Q_INT8>(a, b, (u - wf) * rows, tpw, nF, nQ, sm_t, sm_cs);
  else chunk_scores<D, KT, Q_INT4>(a, b, (u - wf) * rows, tpw, nF, nQ, sm_t, sm_cs);
}

// ---- finish: global softmax statistics, scores, output ------------------------------------------------------
// Global (m, 1/l) of one query head out of the ns split partials at src (stride 2 * G floats), up to N of them with all
// loads in flight together.  A sequence with no live position at all (every position evicted by a forced plan) has
// m = -inf, l = 0 in every split: its output is defined as zero, not 0/0.
template <int G, int N>
__device__ __forceinline__ void merge_stats_n(const float* __restrict__ src, int ns, float& mm, float& ll) {
  float mv[N], lv[N];
#pragma unroll
  for (int k = 0; k < N; ++k) {
    mv[k] = k < ns ? src[k * 2 * G] : -INFINITY;
    lv[k] = k < ns ? src[k * 2 * G + G] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < N; ++k) mm = fmaxf(mm, mv[k]);
  if (mm > -INFINITY) {
#pragma unroll
    for (int k = 0; k < N; ++k) ll = fmaf(lv[k], __builtin_amdgcn_exp2f((mv[k] - mm) * LOG2E), ll);
  }
}
template <int G>
__device__ __forceinline__ void merge_stats(const float* __restrict__ src, int ns, float& m, float& il) {
  float mm = -INFINITY, ll = 0.f;
  if (ns == 1) {
    mm = src[0]; ll = src[G];
  } else if (ns <= 4) {
    merge_stats_n<G, 4>(src, ns, mm, ll);
  } else if (ns <= 8) {
    merge_stats_n<G, 8>(src, ns, mm, ll);
  } else if (ns <= 16) {
    merge_stats_n<G, 16>(src, ns, mm, ll);
  } else {
#pragma unroll 8
    for (int k = 0; k < ns; ++k) mm = fmaxf(mm, src[k * 2 * G]);
    if (mm > -INFINITY) {
#pragma unroll 8
      for (int k = 0; k < ns; ++k) ll = fmaf(src[k * 2 * G + G], __builtin_amdgcn_exp2f((src[k * 2 * G] - mm) * LOG2E), ll);
    }
  }
  m = mm > -INFINITY ? mm : 0.f;
  il = ll > 0.f ? 1.0f / ll : 0.f;
}

// Grid (64-entry tiles + output workgroups, B); a launch finishes the a.nl layers its attention launch served.
// Tile workgroups: 64 list entries; thread (e, hg, ls) sums the softmax weights of entry e over kv heads hg, hg+4, ...
// (all G members of each) for layers ls, ls + LSN, ...; the four partial sums of a layer are added in the order hg = 0..3
// and the layers into the score in layer order, so a whole step and per-layer calls give the same bits.  Latency-bound:
// the logits of a thread's first XP layers are requested before anything they do not depend on, and a step's launch has
// four times the threads, so that the (m, l) merges of all its layers are one round trip.
// Output workgroups: 256 threads per (layer, query head).
template <bool STEP>
struct FinGeo {
  static constexpr int LSN = STEP ? 4 : 1;          // layers in parallel
  static constexpr int NT = 256 * LSN;
  static constexpr int XP = STEP ? 3 : 1;
  static constexpr int LB = STEP ? 32 : 1;          // layers per pass, at most
  static constexpr int NST = STEP ? 2048 : 128;     // (layer, head) statistics per pass, at most
  static constexpr int HPG = STEP ? 4 : 1;          // (layer, head) outputs per 256-thread group
};
template <int D, int G, bool STEP>
__global__ __launch_bounds__(FinGeo<STEP>::NT) void k_attn_finish(const AttnArgs a, int n_tiles) {
  using FG = FinGeo<STEP>;
  constexpr int LSN = FG::LSN, NT = FG::NT, XP = FG::XP;
  __shared__ float2 sm_st[FG::NST];                         // (m, 1/l) of every (layer, head) of the pass
  __shared__ float sm_part[(FG::LB > LSN * FG::HPG ? FG::LB : LSN * FG::HPG) * 256];
  const int t = threadIdx.x, b = blockIdx.y, ns = a.S_total;
  const size_t kv_ml = (size_t)ns * 2 * G;                  // statistics of one (layer, sequence, kv head)
  if ((int)blockIdx.x < n_tiles) {
    int nF = a.nF[b & (ATTN_ARG_SEQS - 1)], nQ = a.nQ[b & (ATTN_ARG_SEQS - 1)], nS;     // asked for beside B, not behind it
    if (a.B > ATTN_ARG_SEQS) { nF = a.cnt[b * CNT_N + C_NF] - a.trim; nQ = a.cnt[b * CNT_N + C_NQ]; }
    nS = a.s_pos ? a.cnt[b * CNT_N + C_NS] : 0;
    // logits columns: F tiles, Q tiles, then (streamed T1) the T1 list's tiles
    const int cf = (nF + TB - 1) / TB, cq = (nQ + TB - 1) / TB;
    if ((int)blockIdx.x * 64 >= (nS > 0 ? (cf + cq) * TB + nS : cf * TB + nQ)) return;
    const int e = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), hg = wv & 3, ls = wv >> 2;
    const int j = blockIdx.x * 64 + e;
    const bool in_f = j < nF, in_q = j >= cf * TB && j - cf * TB < nQ, in_s = j >= (cf + cq) * TB && j - (cf + cq) * TB < nS;
    const bool live = in_f || in_q || in_s;
    int pos = -1;
    if (in_f) pos = a.f_pos[(size_t)b * a.Nmax + j];
    else if (in_q) pos = a.q_pos[(size_t)b * a.Nmax + (j - cf * TB)];
    else if (in_s) pos = a.s_pos[(size_t)b * a.Nmax + (j - (cf + cq) * TB)];
    float score = 0.f;
    // A logit's weight: the matrix cores' waves leave unscaled logits, the others scaled ones.  (A branch on the rows' type in
    // its place costs a call 0.4 us: binary32 rows at a head_dim and group size of the matrix cores' have the exponent's
    // remainder put back in too, for 0.1 us.)
    const float xscale = split_on_matrix(D, G, a.q_es) ? a.softmax_scale : 1.0f;
    const auto weight = [&](float x, const float2& st) {
      if constexpr (split_on_matrix(D, G, 2)) return exp_le0(fmaf(x, xscale, -st.x)) * st.y;
      else return __builtin_amdgcn_exp2f((x - st.x) * LOG2E) * st.y;
    };
    const float pen = a.red ? a.red_w * (float)G / (float)(nF + nQ + nS) : 0.f;
    const int per_pass = STEP ? (FG::NST / a.Hq < FG::LB ? FG::NST / a.Hq : FG::LB) : 1;
    for (int l0 = 0; l0 < a.nl; l0 += per_pass) {
      const int nb = a.nl - l0 < per_pass ? a.nl - l0 : per_pass;
      float x0[XP][G];
#pragma unroll
      for (int q = 0; q < XP; ++q)
        if (ls + q * LSN < nb) {
          const float* xr = a.xs + xs_at(a, (l0 + ls + q * LSN) * a.B + b, hg * G, j);
#pragma unroll
          for (int g = 0; g < G; ++g) x0[q][g] = (live && hg < a.Hkv) ? xr[(size_t)g * a.xs_stride] : 0.f;
        }
      if (l0 == 0 && wv == 0 && live) score = a.score[(size_t)b * a.Nmax + pos];
      for (int i = t; i < nb * a.Hq; i += NT) {
        const int u = STEP ? i / a.Hq : 0, hq = i - u * a.Hq, kvh = hq / G, g = hq % G;
        float m, il;
        merge_stats<G>(a.part_ml + ((size_t)((l0 + u) * a.B + b) * a.Hkv + kvh) * kv_ml + g, ns, m, il);
        sm_st[i] = make_float2(m, il);
      }
      __syncthreads();
      auto layer_sum = [&](int u, const float (&xf)[G], bool have) {
        const int bl = (l0 + u) * a.B + b;
        float acc = 0.f;
        if (live) {
          for (int kvh = hg; kvh < a.Hkv; kvh += 4) {
            float x[G];
#pragma unroll
            for (int g = 0; g < G; ++g) x[g] = (have && kvh == hg) ? xf[g] : a.xs[xs_at(a, bl, kvh * G + g, j)];
            const float2* stt = sm_st + u * a.Hq + kvh * G;
            if (a.vnorm) {
              // value-aware scorer: the group's weights times the norm of the value row its heads read
              float w = 0.f;
#pragma unroll
              for (int g = 0; g < G; ++g) w += weight(x[g], stt[g]);
              acc = fmaf(w, a.vnorm[((size_t)bl * a.Hkv + kvh) * a.Nmax + pos], acc);
            } else {
#pragma unroll
              for (int g = 0; g < G; ++g) acc += weight(x[g], stt[g]);
            }
            // redundancy-penalised scorers: the G heads of the group each take red_w * rho / (positions attended) off
            if (a.red) acc = fmaf(-pen, a.red[((size_t)bl * a.Hkv + kvh) * a.Nmax + pos], acc);
          }
        }
        sm_part[(u * 4 + hg) * 64 + e] = acc;
      };
#pragma unroll
      for (int q = 0; q < XP; ++q)
        if (ls + q * LSN < nb) layer_sum(ls + q * LSN, x0[q], true);
      if constexpr (STEP)
        for (int u = ls + XP * LSN; u < nb; u += LSN) layer_sum(u, x0[0], false);
      __syncthreads();
      if (wv == 0)
        for (int u = 0; u < nb; ++u) {
          const float* s4 = sm_part + u * 256 + e;
          score = score + a.score_scale * (((s4[0] + s4[64]) + s4[128]) + s4[192]);
        }
      if (STEP && l0 + per_pass < a.nl) __syncthreads();
    }
    if (wv == 0 && live) a.score[(size_t)b * a.Nmax + pos] = score;
  } else {
    // thread (d, sg) of a (layer, head) sums the splits sg, sg+NSG, ... of output element d, then the NSG partial sums
    // are added in the fixed order sg = 0, 1, ...
    constexpr int NSG = 256 / D;
    constexpr int HPG = FG::HPG;                            // (layer, head)s per 256-thread group, their loads in flight together
    const int r0 = ((blockIdx.x - n_tiles) * LSN + (t >> 8)) * HPG, tl = t & 255;
    const int d = tl % D, sg = tl / D;
    float il[HPG], acc[HPG];
#pragma unroll
    for (int q = 0; q < HPG; ++q) {
      const int r = r0 + q;
      il[q] = 0.f; acc[q] = 0.f;
      if (r < a.nl * a.Hq) {
        const int li = STEP ? r / a.Hq : 0, hq = r - li * a.Hq, kvh = hq / G, h = hq % G, bl = li * a.B + b;
        const float* pm = a.part_ml + ((size_t)bl * a.Hkv + kvh) * kv_ml + h;
        const float* pob = a.part_o + ((size_t)(bl * a.Hkv + kvh) * ns * G) * D + h * D + d;
        float mg;
        merge_stats<G>(pm, ns, mg, il[q]);
#pragma unroll 8
        for (int k = sg; k < ns; k += NSG)
          acc[q] = fmaf(__builtin_amdgcn_exp2f((pm[k * 2 * G] - mg) * LOG2E), pob[(size_t)k * G * D], acc[q]);
      }
    }
    float* sp = sm_part + (t >> 8) * (256 * HPG) + sg * D + d;
#pragma unroll
    for (int q = 0; q < HPG; ++q) sp[q * 256] = acc[q];
    __syncthreads();
    if (sg == 0) {
#pragma unroll
      for (int q = 0; q < HPG; ++q) {
        const int r = r0 + q;
        if (r >= a.nl * a.Hq) continue;
        float tot = acc[q];
#pragma unroll
        for (int g2 = 1; g2 < NSG; ++g2) tot += sp[q * 256 + g2 * D];
        tot *= il[q];
        const int li = STEP ? r / a.Hq : 0, hq = r - li * a.Hq;
        const size_t oi = ((size_t)(li * a.B + b) * a.o_bs + hq) * D + d;
        if (a.out_kind == KT_BF16) ((uint16_t*)a.out)[oi] = f32_to_bf16(tot);
        else if (a.out_kind == KT_F16) ((_Float16*)a.out)[oi] = (_Float16)tot;    // round to nearest even
        else ((float*)a.out)[oi] = tot;
      }
    }
  }
}

// ---- finish for several query tokens per sequence whose logits were written (one launch served n_q * cq of them) ------
// Grid (64-entry slots of the last token's lists + output workgroups, B).  Slot workgroups: every list entry gets the
// weights of the queries added in query order (what single-token calls would have done, with the same arithmetic per
// query: wave (hg, ls) sums kv heads hg, hg+4, ... for queries ls, ls+LSN, ..., the four partial sums are added in the order
// hg = 0..3).  Query jt does not see the last n_q - 1 - jt entries of list F; its Q-list logits start where its F tiles
// end (16-bit rows, all in one column group: where the last token's do).  Latency-bound like k_attn_finish and built like it: the first logits are requested before the statistics, LSN
// queries go side by side (256 threads each).  The other workgroups merge the splits of LSN * hpg (query, head)s into out,
// hpg of them one after the other in a thread: two where the merge is one round of loads, one where it is a chain (more
// than 16 splits).
constexpr int CHUNK_HPG = 2;
template <int D, int G, int LSN>
__global__ __launch_bounds__(LSN * 256) void k_attn_finish_chunk(const AttnArgs a, int n_tiles, int hpg) {
  constexpr int XP = LSN == 1 ? 4 : 2;
  extern __shared__ __attribute__((aligned(8))) float sm_dyn[];    // statistics [nq][Hq], then partial sums [nq][4][64] / [LSN][HPG][256]
  const int t = threadIdx.x, b = blockIdx.y, nq = a.n_q * a.cq, ns = a.S_total;
  float2* sm_st = (float2*)sm_dyn;
  float* sm_part = sm_dyn + 2 * nq * a.Hq;
  const size_t kv_ml = (size_t)ns * 2 * G;
  if ((int)blockIdx.x < n_tiles) {
    int nF = a.nF[b & (ATTN_ARG_SEQS - 1)], nQ = a.nQ[b & (ATTN_ARG_SEQS - 1)];
    if (a.B > ATTN_ARG_SEQS) { nF = a.cnt[b * CNT_N + C_NF] - a.trim; nQ = a.cnt[b * CNT_N + C_NQ]; }
    const int cf = (nF + TB - 1) / TB;                       // F tiles of the last query (the longest list)
    if ((int)blockIdx.x * 64 >= cf * TB + nQ) return;
    const int e = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), hg = wv & 3, ls = wv >> 2;
    const int sl = blockIdx.x * 64 + e;                     // slot in the last query's layout
    const bool is_f = sl < nF, is_q = sl >= cf * TB && sl - cf * TB < nQ;
    auto sees = [&](int jt) { return is_q || (is_f && sl < nF - (nq - 1 - jt)); };   // wave-divergent at most in a list's last tile
    auto column = [&](int jt) {                             // binary32: F tiles in the query's own layout
      const int cfz = a.cq > 1 ? cf : (nF - (nq - 1 - jt) + TB - 1) / TB;
      return is_q ? cfz * TB + (sl - cf * TB) : sl;
    };
    float x0[XP][G];
#pragma unroll
    for (int q = 0; q < XP; ++q) {
      const int jt = ls + LSN * q;
      if (jt < nq) {
        const bool in = hg < a.Hkv && sees(jt);
        const float* xr = a.xs + xs_at(a, b * nq + jt, hg * G, column(jt));
#pragma unroll
        for (int g = 0; g < G; ++g) x0[q][g] = in ? xr[(size_t)g * a.xs_stride] : 0.f;
      }
    }
    int pos = -1;
    if (is_f) pos = a.f_pos[(size_t)b * a.Nmax + sl];
    else if (is_q) pos = a.q_pos[(size_t)b * a.Nmax + (sl - cf * TB)];
    // global (m, 1/l) of every (query, head) of this sequence
    for (int i = t; i < nq * a.Hq; i += LSN * 256) {
      const int jt = i / a.Hq, hq = i - jt * a.Hq, kvh = hq / G, g = hq % G;
      float m, il;
      merge_stats<G>(a.part_ml + (size_t)((b * nq + jt) * a.Hkv + kvh) * kv_ml + g, ns, m, il);
      sm_st[i] = make_float2(m, il);
    }
    float score = (wv == 0 && pos >= 0) ? a.score[(size_t)b * a.Nmax + pos] : 0.f;
    __syncthreads();
    auto token_sum = [&](int jt, const float (&xf)[G], bool have) {
      float acc = 0.f;
      if (sees(jt)) {
        const float pen = a.red ? a.red_w * (float)G / (float)(nF - (nq - 1 - jt) + nQ) : 0.f;
        const int col = column(jt);
        for (int kvh = hg; kvh < a.Hkv; kvh += 4) {
          float x[G];
#pragma unroll
          for (int g = 0; g < G; ++g) x[g] = (have && kvh == hg) ? xf[g] : a.xs[xs_at(a, b * nq + jt, kvh * G + g, col)];
          const float2* stt = sm_st + jt * a.Hq + kvh * G;
          if (a.vnorm) {
            float w = 0.f;
#pragma unroll
            for (int g = 0; g < G; ++g) w += __builtin_amdgcn_exp2f((x[g] - stt[g].x) * LOG2E) * stt[g].y;
            acc = fmaf(w, a.vnorm[((size_t)b * a.Hkv + kvh) * a.Nmax + pos], acc);
          } else {
#pragma unroll
            for (int g = 0; g < G; ++g) acc += __builtin_amdgcn_exp2f((x[g] - stt[g].x) * LOG2E) * stt[g].y;
          }
          if (a.red) acc = fmaf(-pen, a.red[((size_t)b * a.Hkv + kvh) * a.Nmax + pos], acc);
        }
      }
      sm_part[(jt * 4 + hg) * 64 + e] = acc;
    };
#pragma unroll
    for (int q = 0; q < XP; ++q)
      if (ls + LSN * q < nq) token_sum(ls + LSN * q, x0[q], true);
    for (int jt = ls + LSN * XP; jt < nq; jt += LSN) token_sum(jt, x0[0], false);
    __syncthreads();
    if (wv == 0 && pos >= 0) {
      for (int jt = 0; jt < nq; ++jt) {
        const float* s4 = sm_part + jt * 256 + e;
        if (sees(jt)) score = score + a.score_scale * (((s4[0] + s4[64]) + s4[128]) + s4[192]);
      }
      a.score[(size_t)b * a.Nmax + pos] = score;
    }
  } else {
    constexpr int NSG = 256 / D, HPG = CHUNK_HPG;
    const int r0 = ((blockIdx.x - n_tiles) * LSN + (t >> 8)) * hpg, tl = t & 255;
    const int d = tl % D, sg = tl / D;
    float il[HPG], acc[HPG];
#pragma unroll
    for (int q = 0; q < HPG; ++q) {
      const int r = r0 + q;
      il[q] = 0.f; acc[q] = 0.f;
      if (q < hpg && r < nq * a.Hq) {
        const int jt = r / a.Hq, hq = r - jt * a.Hq, kvh = hq / G, h = hq % G;
        const float* pm = a.part_ml + (size_t)((b * nq + jt) * a.Hkv + kvh) * kv_ml + h;
        const float* pob = a.part_o + ((size_t)((b * nq + jt) * a.Hkv + kvh) * ns * G) * D + h * D + d;
        float mg;
        merge_stats<G>(pm, ns, mg, il[q]);
#pragma unroll 4
        for (int k = sg; k < ns; k += NSG)
          acc[q] = fmaf(__builtin_amdgcn_exp2f((pm[k * 2 * G] - mg) * LOG2E), pob[(size_t)k * G * D], acc[q]);
      }
    }
    float* sp = sm_part + (t >> 8) * (256 * HPG) + sg * D + d;
#pragma unroll
    for (int q = 0; q < HPG; ++q) sp[q * 256] = acc[q];
    __syncthreads();
    if (sg == 0) {
#pragma unroll
      for (int q = 0; q < HPG; ++q) {
        const int r = r0 + q;
        if (q >= hpg || r >= nq * a.Hq) continue;
        float tot = acc[q];
#pragma unroll
        for (int g2 = 1; g2 < NSG; ++g2) tot += sp[q * 256 + g2 * D];
        tot *= il[q];
        const int jt = r / a.Hq, hq = r - jt * a.Hq;
        const size_t oi = ((size_t)b * a.o_bs + (size_t)jt * a.Hq + hq) * D + d;
        if (a.out_kind == KT_BF16) ((uint16_t*)a.out)[oi] = f32_to_bf16(tot);
        else if (a.out_kind == KT_F16) ((_Float16*)a.out)[oi] = (_Float16)tot;
        else ((float*)a.out)[oi] = tot;
      }
    }
  }
}

#if !defined(TKV_ATTN_PART) || TKV_ATTN_PART == 4
// ---- finish of a whole-pair step launch: the rows' weights summed over kv heads and layers into the scores ----------
// Grid (64-column tiles, B), a wave per layer up to 16: wave w sums the kv heads of layers w, w + 16, ...; the layers are
// then added into the score in layer order, so that it does not matter how a step's layers are grouped into launches.
__global__ __launch_bounds__(1024) void k_step_scores(const AttnArgs a, int tr) {
  __shared__ float tot[MAX_LAYERS_PER_LAUNCH * 64];
  const int b = blockIdx.y, t = threadIdx.x, e = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), c = blockIdx.x * 64 + e;
  int nF, nQ;
  if (a.B <= ATTN_ARG_SEQS) { nF = a.nF[b]; nQ = a.nQ[b]; }
  else { nF = a.cnt[b * CNT_N + C_NF]; nQ = a.cnt[b * CNT_N + C_NQ]; }
  const int colq = (nF + tr - 1) / tr * tr;
  if ((int)blockIdx.x * 64 >= colq + nQ) return;
  const bool live = c < nF || (c >= colq && c < colq + nQ);
  for (int l = wv; l < a.nl; l += blockDim.x >> 6) {
    const float* src = a.sc + ((size_t)(l * a.B + b) * a.Hkv) * a.sc_stride + c;
    float s = 0.f;
    if (live) {
#pragma unroll 8
      for (int k = 0; k < a.Hkv; ++k) s += src[(size_t)k * a.sc_stride];
    }
    tot[l * 64 + e] = s;
  }
  int pos = 0;
  float score = 0.f;
  if (wv == 0 && live) {
    pos = c < nF ? a.f_pos[(size_t)b * a.Nmax + c] : a.q_pos[(size_t)b * a.Nmax + (c - colq)];
    score = a.score[(size_t)b * a.Nmax + pos];
  }
  __syncthreads();
  if (wv == 0 && live) {
    for (int l = 0; l < a.nl; ++l) score = score + a.score_scale * tot[l * 64 + e];
    a.score[(size_t)b * a.Nmax + pos] = score;
  }
}

// The same where the last pairs were walked in parts: their weights are made here, from the logits and the merged statistics of
// the parts, with the arithmetic of k_attn_step, and the last workgroups merge their outputs.  Grid (tiles of COLS columns +
// output workgroups, B).  Bound by latency: a split pair is G loads a column where a whole one is one, and one sequence of 1422
// tokens has 23 tiles of 64 columns for 256 compute units.  There a wave's lanes are 16 columns of four kv heads, two layers
// at a time (6.3 us); where the tiles fill the chip they are 64 columns, four kv heads one after the other with their loads in
// flight together (8 x 2081, 28 layers, four kv heads: 19.7 us with 16).  Either way the kv heads are added one by one, as
// k_step_scores and k_call_scores do.
template <int G, int COLS>
__global__ __launch_bounds__(1024) void k_step_scores_parts(const AttnArgs a, int tr, int n_ct, int D) {
  extern __shared__ float2 sm_st[];                      // (m, 1/l) of every head of the layers with a split pair, from layer l0 on
  __shared__ float tot[MAX_LAYERS_PER_LAUNCH * COLS];
  const int b = blockIdx.y, t = threadIdx.x;
  if ((int)blockIdx.x >= n_ct) {
    const size_t i = ((size_t)(blockIdx.x - n_ct) * gridDim.y + b) * blockDim.x + t, total = (size_t)(a.nl * a.B - a.whole_rows) * a.Hkv * G * D;
    if (i >= total) return;
    const int e = (int)(i % ((size_t)G * D)), h = e / D, pair = a.whole_rows * a.Hkv + (int)(i / ((size_t)G * D));
    const size_t sp = (size_t)(pair + a.tail0) * a.S;
    const float* pm = a.part_ml + sp * 2 * G + h;
    float m, il, acc = 0.f;
    merge_stats<G>(pm, a.S, m, il);
#pragma unroll 8
    for (int k = 0; k < a.S; ++k)
      acc = fmaf(__builtin_amdgcn_exp2f((pm[k * 2 * G] - m) * LOG2E), a.part_o[(sp + k) * G * D + e], acc);
    acc *= il;
    const int bl = pair / a.Hkv, kvh = pair - bl * a.Hkv;
    const size_t oi = ((size_t)bl * a.o_bs + kvh * G) * D + e;
    if (a.out_kind == KT_BF16) ((uint16_t*)a.out)[oi] = f32_to_bf16(acc);
    else if (a.out_kind == KT_F16) ((_Float16*)a.out)[oi] = (_Float16)acc;    // round to nearest even
    else ((float*)a.out)[oi] = acc;
    return;
  }
  int nF, nQ;
  if (a.B <= ATTN_ARG_SEQS) { nF = a.nF[b]; nQ = a.nQ[b]; }
  else { nF = a.cnt[b * CNT_N + C_NF]; nQ = a.cnt[b * CNT_N + C_NQ]; }
  const int colq = (nF + tr - 1) / tr * tr;
  if ((int)blockIdx.x * COLS >= colq + nQ) return;
  constexpr int NSG = 64 / COLS, KK = 4 / NSG, LB = NSG == 1 ? 1 : 2;   // kv heads side by side and one after the other, layers at a time
  const int e = t % COLS, sg = (t % 64) / COLS, wv = __builtin_amdgcn_readfirstlane(t >> 6), nwv = blockDim.x >> 6;
  const int c = blockIdx.x * COLS + e;
  const bool live = c < nF || (c >= colq && c < colq + nQ);
  int pos = 0;
  float score = 0.f;
  if (live) pos = c < nF ? a.f_pos[(size_t)b * a.Nmax + c] : a.q_pos[(size_t)b * a.Nmax + (c - colq)];
  if (live && t < COLS) score = a.score[(size_t)b * a.Nmax + pos];
  const int l0 = a.whole_rows > b ? (a.whole_rows - b + a.B - 1) / a.B : 0;      // the sequence's first layer whose pairs are split
  for (int i = t; i < (a.nl - l0) * a.Hq; i += blockDim.x) {
    const int l = l0 + i / a.Hq, hq = i % a.Hq, k = hq / G, pair = (l * a.B + b) * a.Hkv + k;
    float m, il;
    merge_stats<G>(a.part_ml + (size_t)(pair + a.tail0) * a.S * 2 * G + (hq - k * G), a.S, m, il);
    sm_st[i] = make_float2(m, il);
  }
  __syncthreads();
  const float pen = a.red ? a.red_w * (float)G / (float)(nF + nQ) : 0.f;
  for (int lb = wv; lb < a.nl; lb += LB * nwv) {
    float s[LB];
#pragma unroll
    for (int q = 0; q < LB; ++q) s[q] = 0.f;
    for (int k0 = 0; k0 < a.Hkv; k0 += 4) {
      float x[LB][KK][G], w[LB][KK];
      bool parts[LB][KK];
#pragma unroll
      for (int q = 0; q < LB; ++q)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const int l = lb + q * nwv, k = k0 + kk + sg, pair = (l * a.B + b) * a.Hkv + k;
          const bool have = l < a.nl && k < a.Hkv;
          parts[q][kk] = have && l >= l0;
          w[q][kk] = 0.f;
          if (live && have && !parts[q][kk]) w[q][kk] = a.sc[(size_t)pair * a.sc_stride + c];
          if (live && parts[q][kk]) {
            const float* src = a.xt + (size_t)(pair + a.tail0) * G * a.sc_stride + c;
#pragma unroll
            for (int g = 0; g < G; ++g) x[q][kk][g] = src[(size_t)g * a.sc_stride];
          }
        }
#pragma unroll
      for (int q = 0; q < LB; ++q) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          if (live && parts[q][kk]) {
            const int l = lb + q * nwv, k = k0 + kk + sg;
            const size_t pr = (size_t)(l * a.B + b) * a.Hkv + k;
            const float2* st = sm_st + (l - l0) * a.Hq + k * G;
#pragma unroll
            for (int g = 0; g < G; ++g) w[q][kk] += exp_le0(fmaf(x[q][kk][g], a.softmax_scale, -st[g].x)) * st[g].y;
            if (a.vnorm) w[q][kk] *= a.vnorm[pr * a.Nmax + pos];
            if (a.red) w[q][kk] = fmaf(-pen, a.red[pr * a.Nmax + pos], w[q][kk]);
          }
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (k0 + j < a.Hkv) s[q] += NSG == 1 ? w[q][j % KK] : __shfl(w[q][0], COLS * j + e);
      }
    }
#pragma unroll
    for (int q = 0; q < LB; ++q)
      if (sg == 0 && lb + q * nwv < a.nl) tot[(lb + q * nwv) * COLS + e] = s[q];
  }
  __syncthreads();
  if (t < COLS && live) {
    for (int l = 0; l < a.nl; ++l) score = score + a.score_scale * tot[l * COLS + e];
    a.score[(size_t)b * a.Nmax + pos] = score;
  }
}

// The same for one layer: nothing to add up but the kv heads, so a thread takes two columns and has all their loads in
// flight (64 sequences of 16384 tokens, 17 MB: 22 us with a wave per 64 columns as above).
__global__ __launch_bounds__(256) void k_call_scores(const AttnArgs a, int tr) {
  const int b = blockIdx.y;
  int nF = a.nF[b & (ATTN_ARG_SEQS - 1)], nQ = a.nQ[b & (ATTN_ARG_SEQS - 1)];
  if (a.B > ATTN_ARG_SEQS) { nF = a.cnt[b * CNT_N + C_NF]; nQ = a.cnt[b * CNT_N + C_NQ]; }
  const int colq = (nF + tr - 1) / tr * tr;
  int pos[2];
  float s[2] = {0.f, 0.f};
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int c = blockIdx.x * 512 + u * 256 + threadIdx.x;
    pos[u] = -1;
    if (c < nF) pos[u] = a.f_pos[(size_t)b * a.Nmax + c];
    else if (c >= colq && c < colq + nQ) pos[u] = a.q_pos[(size_t)b * a.Nmax + (c - colq)];
    if (c < nF || (c >= colq && c < colq + nQ)) {
      const float* src = a.sc + (size_t)b * a.Hkv * a.sc_stride + c;
#pragma unroll 8
      for (int k = 0; k < a.Hkv; ++k) s[u] += src[(size_t)k * a.sc_stride];
    }
  }
  float score[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) score[u] = pos[u] >= 0 ? a.score[(size_t)b * a.Nmax + pos[u]] : 0.f;
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (pos[u] >= 0) a.score[(size_t)b * a.Nmax + pos[u]] = score[u] + a.score_scale * s[u];
}
#endif

// ---- dispatch ----------------------------------------------------------------------------------------------
// The file is compiled once per part (TKV_ATTN_PART = 0..3, 5, 6: one (head_dim, KV dtype) pair of attn_tiered each,
// 4: attn_finish and the launchers), so the parts build in parallel; without the macro it is one translation unit.
#if defined(TKV_ATTN_PART)
#define TKV_HAS_PART(p) (TKV_ATTN_PART == (p))
#else
#define TKV_HAS_PART(p) 1
#endif

#define TKV_DISPATCH_G(FN, D_, BF_, ...)                    \
  switch (G) {                                              \
    case 1: return FN<D_, 1, BF_>(__VA_ARGS__);             \
    case 2: return FN<D_, 2, BF_>(__VA_ARGS__);             \
    case 3: return FN<D_, 3, BF_>(__VA_ARGS__);             \
    case 4: return FN<D_, 4, BF_>(__VA_ARGS__);             \
    case 5: return FN<D_, 5, BF_>(__VA_ARGS__);             \
    case 6: return FN<D_, 6, BF_>(__VA_ARGS__);             \
    case 7: return FN<D_, 7, BF_>(__VA_ARGS__);             \
    case 8: return FN<D_, 8, BF_>(__VA_ARGS__);             \
    default: return hipErrorInvalidValue;                   \
  }

// With a pair of events the launch is timed by the dispatch's own begin / end timestamps (no bracket overhead).
template <int D, int G, int KT>
static hipError_t run_tiered(const AttnArgs& a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  // one query token per workgroup: the vector kernel, G dot products per row
  const dim3 grid(a.S, a.Hkv, a.B * a.n_q * a.nl);
  constexpr int threads = KernelGeo<D, G, KT>::NW * 64;
  if (ev0 && ev1) hipExtLaunchKernelGGL((k_attn_tiered<D, G, KT>), grid, dim3(threads), 0, st, ev0, ev1, 0, a);
  else hipLaunchKernelGGL((k_attn_tiered<D, G, KT>), grid, dim3(threads), 0, st, a);
  return hipGetLastError();
}
// Several query tokens as columns of one workgroup (16-bit rows): a (rows x D) by (D x columns) contraction, on the matrix
// cores; then the scores and the outputs.
// Tiles per workgroup of the score launch: one workgroup for every compute unit (of 256) but some 32 for the outputs, as far
// as the LDS has room.
static int chunk_tiles_per_wg(const AttnArgs& a, int D, int tiles) {
  int tpw = (int)std::min<int64_t>(CS_THREADS / CS_ROWS, ((int64_t)(tiles + 1) * a.B + 223) / 224);
  while (tpw > 1 && chunk_scores_lds(a.Hq, a.Hkv, a.cq, a.G, tpw) > cs_lds(D)) --tpw;
  return tpw < 1 ? 1 : tpw;
}
template <int D, int KT>
static hipError_t run_chunk(const AttnArgs& a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const int ncol = a.cq * a.G, ncb = a.xs_stride ? chunk_blocks(ncol) : 2;
  const dim3 grid(a.S, a.Hkv, a.B * a.groups);
  if (a.cq < 2 || a.cq > CHUNK_TOKENS || a.groups != (ncol + 16 * ncb - 1) / (16 * ncb)) return hipErrorInvalidValue;
  if (a.xs_stride && a.groups > 1) return hipErrorInvalidValue;
  const auto kernel = !a.xs_stride ? k_attn_tiered_mc<D, KT, 2, false> : ncb == 1 ? k_attn_tiered_mc<D, KT, 1, true> : k_attn_tiered_mc<D, KT, 2, true>;
  if (ev0 && ev1) hipExtLaunchKernelGGL(kernel, grid, dim3(MC_WAVES * 64), 0, st, ev0, ev1, 0, a);
  else hipLaunchKernelGGL(kernel, grid, dim3(MC_WAVES * 64), 0, st, a);
  if (a.xs_stride) return hipGetLastError();             // the logits are written: launch_attn_finish_chunk ends the call
  if (const hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  const int tiles = a.n_tiles * (64 / CS_ROWS), tpw = chunk_tiles_per_wg(a, D, tiles);
  const int n_wgs = (tiles + tpw - 1) / tpw + 1;         // (list F and list Q both end in a partly filled run)
  // output workgroups: the compute units left over, with at least a row and at most 16 rows for every D threads
  const int rows = a.Hkv * ncol, par = CS_THREADS / D;
  const int n_out = a.S > 4 ? rows : std::max((rows + 16 * par - 1) / (16 * par), std::min((rows + par - 1) / par, 256 / a.B - n_wgs));
  hipLaunchKernelGGL((k_attn_chunk_scores<D, KT>), dim3(n_wgs + n_out, a.B), dim3(CS_THREADS), chunk_scores_lds(a.Hq, a.Hkv, a.cq, a.G, tpw), st, a, n_wgs, tpw);
  return hipGetLastError();
}
template <int D, int G, int KT>
static hipError_t run_step(const AttnArgs& a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if constexpr (KT == KT_F32) {
    return hipErrorInvalidValue;
  } else {
    const dim3 grid(a.Hkv, a.whole_rows + (a.nl * a.B - a.whole_rows) * a.S);
    if constexpr (step_on_vector(D, G, 0)) {
      if (a.vec) {
        if (ev0 && ev1) hipExtLaunchKernelGGL((k_attn_step<D, G, KT, true>), grid, dim3(512), 0, st, ev0, ev1, 0, a);
        else hipLaunchKernelGGL((k_attn_step<D, G, KT, true>), grid, dim3(512), 0, st, a);
        return hipGetLastError();
      }
    }
    if (ev0 && ev1) hipExtLaunchKernelGGL((k_attn_step<D, G, KT, false>), grid, dim3(512), 0, st, ev0, ev1, 0, a);
    else hipLaunchKernelGGL((k_attn_step<D, G, KT, false>), grid, dim3(512), 0, st, a);
    return hipGetLastError();
  }
}
template <int D, int KT>
hipError_t tiered_by_group(const AttnArgs& a, int G, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1);
#define TKV_DEFINE_PART(D_, BF_)                                                                                   \
  template <>                                                                                                      \
  hipError_t tiered_by_group<D_, BF_>(const AttnArgs& a, int G, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {  \
    if (a.groups) {                                                                                                \
      if constexpr (BF_ != KT_F32) return run_chunk<D_, BF_>(a, st, ev0, ev1);                                     \
      return hipErrorInvalidValue;                                                                                 \
    }                                                                                                              \
    if (a.sc) { TKV_DISPATCH_G(run_step, D_, BF_, a, st, ev0, ev1) }                                               \
    TKV_DISPATCH_G(run_tiered, D_, BF_, a, st, ev0, ev1)                                                           \
  }
#if TKV_HAS_PART(0)
TKV_DEFINE_PART(128, KT_BF16)
#endif
#if TKV_HAS_PART(1)
TKV_DEFINE_PART(128, KT_F32)
#endif
#if TKV_HAS_PART(2)
TKV_DEFINE_PART(64, KT_BF16)
#endif
#if TKV_HAS_PART(3)
TKV_DEFINE_PART(64, KT_F32)
#endif
#if TKV_HAS_PART(5)
TKV_DEFINE_PART(128, KT_F16)
#endif
#if TKV_HAS_PART(6)
TKV_DEFINE_PART(64, KT_F16)
#endif

#if TKV_HAS_PART(4)
template <> hipError_t tiered_by_group<128, KT_BF16>(const AttnArgs&, int, hipStream_t, hipEvent_t, hipEvent_t);
template <> hipError_t tiered_by_group<128, KT_F32>(const AttnArgs&, int, hipStream_t, hipEvent_t, hipEvent_t);
template <> hipError_t tiered_by_group<128, KT_F16>(const AttnArgs&, int, hipStream_t, hipEvent_t, hipEvent_t);
template <> hipError_t tiered_by_group<64, KT_BF16>(const AttnArgs&, int, hipStream_t, hipEvent_t, hipEvent_t);
template <> hipError_t tiered_by_group<64, KT_F32>(const AttnArgs&, int, hipStream_t, hipEvent_t, hipEvent_t);
template <> hipError_t tiered_by_group<64, KT_F16>(const AttnArgs&, int, hipStream_t, hipEvent_t, hipEvent_t);

template <int D, int G, bool STEP>
static hipError_t run_finish_layers(const AttnArgs& a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  using FG = FinGeo<STEP>;
  const int opw = FG::LSN * FG::HPG;
  const dim3 grid(a.n_tiles + (a.nl * a.Hq + opw - 1) / opw, a.B);
  if (ev0 && ev1) hipExtLaunchKernelGGL((k_attn_finish<D, G, STEP>), grid, dim3(FG::NT), 0, st, ev0, ev1, 0, a, a.n_tiles);
  else hipLaunchKernelGGL((k_attn_finish<D, G, STEP>), grid, dim3(FG::NT), 0, st, a, a.n_tiles);
  return hipGetLastError();
}
template <int D, int G, int KT>
static hipError_t run_finish(const AttnArgs& a, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  return a.nl > 1 ? run_finish_layers<D, G, true>(a, st, ev0, ev1) : run_finish_layers<D, G, false>(a, st, ev0, ev1);
}

hipError_t launch_attn_tiered(const AttnArgs& a, int D, int G, int kt, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (D == 128 && kt == KT_BF16) return tiered_by_group<128, KT_BF16>(a, G, st, ev0, ev1);
  if (D == 128 && kt == KT_F32) return tiered_by_group<128, KT_F32>(a, G, st, ev0, ev1);
  if (D == 128 && kt == KT_F16) return tiered_by_group<128, KT_F16>(a, G, st, ev0, ev1);
  if (D == 64 && kt == KT_BF16) return tiered_by_group<64, KT_BF16>(a, G, st, ev0, ev1);
  if (D == 64 && kt == KT_F32) return tiered_by_group<64, KT_F32>(a, G, st, ev0, ev1);
  if (D == 64 && kt == KT_F16) return tiered_by_group<64, KT_F16>(a, G, st, ev0, ev1);
  return hipErrorInvalidValue;
}
int attn_waves_per_group(int D, int elem_bytes, int G) { return split_waves(D, elem_bytes, G); }
int attn_tile_rows(int D, int elem_bytes) { return split_tile_rows(D, elem_bytes); }
int attn_chunk_blocks(int n_cols) { return chunk_blocks(n_cols); }
bool attn_chunk_logits(int n_tokens, int G) { return chunk_logits(n_tokens, G); }
int attn_chunk_waves() { return MC_WAVES; }
int attn_chunk_tile_rows(int D) { return mc_tile_rows(D); }
// Query tokens of a chunk that one launch serves: as many as grid z and, where the score launch is the second one, its LDS have
// room for (128 kv heads at head_dim 128: 16, the most with written logits; the score launch would have room for 11).
int attn_chunk_tokens(int B, int Hq, int Hkv, int D) {
  const int G = Hq / Hkv;
  const auto room = [&](int m) {
    return (int64_t)B * ((m * G + 15) / 16) <= 65535 && (chunk_logits(m, G) || chunk_scores_lds(Hq, Hkv, m, G, 1) <= cs_lds(D));
  };
  int m = CHUNK_TOKENS;
  while (m > 1 && !room(m)) --m;
  return m;
}
int attn_q_waves(int n_waves, int n_f_tiles, int n_q_tiles) { return q_waves(n_waves, n_f_tiles, n_q_tiles); }

static int chunk_hpg(const AttnArgs& a) { return a.S_total <= 16 ? CHUNK_HPG : 1; }
static int chunk_workgroups(const AttnArgs& a, int lsn) {   // per sequence
  const int per_wg = lsn * chunk_hpg(a);
  return a.n_tiles + (a.Hq * a.n_q * a.cq + per_wg - 1) / per_wg;
}
template <int D, int G, int LSN>
static hipError_t run_finish_chunk_n(const AttnArgs& a, hipStream_t st) {
  const int nq = a.n_q * a.cq, lds = nq * a.Hq * 8 + (nq > LSN * CHUNK_HPG ? nq : LSN * CHUNK_HPG) * 1024;   // at most 32 KB
  hipLaunchKernelGGL((k_attn_finish_chunk<D, G, LSN>), dim3(chunk_workgroups(a, LSN), a.B), dim3(LSN * 256), lds, st, a, a.n_tiles, chunk_hpg(a));
  return hipGetLastError();
}
template <int D, int G, int KT>
static hipError_t run_finish_chunk(const AttnArgs& a, hipStream_t st) {
  // Queries side by side.  Many tiles fill the chip by themselves (67 x 8 tiles take 13.0 us with LSN = 4, 11.4 with 1; 34 x 8
  // 9.3 and 10.5).  Two queries have nothing for a third and fourth group of threads.  From three on as many as leave room for
  // the output workgroups beside the tiles (2048 threads per compute unit; 32 sequences of 600 tokens, 12/2 heads, four
  // tokens: 26.6 us a call with LSN = 4, 22.9 with 2; 300 tokens, 28/4 heads: 29.3 with 4, 27.3 with 1), but above eight the
  // queries of a thread one after the other weigh more (300 tokens, 8/8 heads, 13 tokens: 29.8 us with 4, 35.2 with 2).
  const int nq = a.n_q * a.cq;
  const auto fits = [&](int lsn) { return (int64_t)chunk_workgroups(a, lsn) * a.B * lsn <= 256 * 8; };
  if ((int64_t)a.n_tiles * a.B > 384) return run_finish_chunk_n<D, G, 1>(a, st);
  if (nq > 8 || (nq > 2 && fits(4))) return run_finish_chunk_n<D, G, 4>(a, st);
  if (nq <= 2 || fits(2)) return run_finish_chunk_n<D, G, 2>(a, st);
  return run_finish_chunk_n<D, G, 1>(a, st);
}
hipError_t launch_attn_finish_chunk(const AttnArgs& a, int D, int G, hipStream_t st) {
  if (a.n_q < 1 || a.cq < 1 || a.n_q * a.cq > 16 || a.Hq > 128) return hipErrorInvalidValue;
  if (D == 128) { TKV_DISPATCH_G(run_finish_chunk, 128, KT_BF16, a, st) }
  if (D == 64) { TKV_DISPATCH_G(run_finish_chunk, 64, KT_BF16, a, st) }
  return hipErrorInvalidValue;
}

bool attn_step_on_vector(int D, int G, int max_tokens) { return step_on_vector(D, G, max_tokens); }
int attn_step_tile_rows(int D) { return D == 128 ? StepGeo<128, 1>::TR : StepGeo<64, 1>::TR; }
template <int D, int G, int KT>
static int step_cap() { return StepGeo<D, G>::LCAP; }
int attn_step_lds_entries(int D, int G) {
  const auto of_d128 = [&]() -> int { switch (G) { case 1: return step_cap<128, 1, 1>(); case 2: return step_cap<128, 2, 1>(); case 3: return step_cap<128, 3, 1>();
    case 4: return step_cap<128, 4, 1>(); case 5: return step_cap<128, 5, 1>(); case 6: return step_cap<128, 6, 1>(); case 7: return step_cap<128, 7, 1>(); default: return step_cap<128, 8, 1>(); } };
  const auto of_d64 = [&]() -> int { switch (G) { case 1: return step_cap<64, 1, 1>(); case 2: return step_cap<64, 2, 1>(); case 3: return step_cap<64, 3, 1>();
    case 4: return step_cap<64, 4, 1>(); case 5: return step_cap<64, 5, 1>(); case 6: return step_cap<64, 6, 1>(); case 7: return step_cap<64, 7, 1>(); default: return step_cap<64, 8, 1>(); } };
  return D == 128 ? of_d128() : of_d64();
}
template <int G, int COLS>
static hipError_t run_scores_parts_n(const AttnArgs& a, int D, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  const int tr = attn_step_tile_rows(D), threads = 64 * (a.nl < 16 ? a.nl : 16), n_ct = a.n_tiles * (64 / COLS);
  const int rows = a.nl * a.B - a.whole_rows, layers = (rows + a.B - 1) / a.B;    // split rows, layers that have some
  const int64_t per_y = (int64_t)threads * a.B;
  const dim3 grid((unsigned)(n_ct + ((int64_t)rows * a.Hkv * G * D + per_y - 1) / per_y), a.B);
  const size_t lds = (size_t)layers * a.Hq * sizeof(float2);
  if (ev0 && ev1) hipExtLaunchKernelGGL((k_step_scores_parts<G, COLS>), grid, dim3(threads), lds, st, ev0, ev1, 0, a, tr, n_ct, D);
  else hipLaunchKernelGGL((k_step_scores_parts<G, COLS>), grid, dim3(threads), lds, st, a, tr, n_ct, D);
  return hipGetLastError();
}
template <int, int G, int>
static hipError_t run_scores_parts(const AttnArgs& a, int D, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  return a.n_tiles * a.B < 128 ? run_scores_parts_n<G, 16>(a, D, st, ev0, ev1) : run_scores_parts_n<G, 64>(a, D, st, ev0, ev1);
}
hipError_t launch_step_scores(const AttnArgs& a, int D, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (a.nl < 1 || a.nl > MAX_LAYERS_PER_LAUNCH) return hipErrorInvalidValue;
  if (a.whole_rows < a.nl * a.B) {
    const int G = a.Hq / a.Hkv;
    TKV_DISPATCH_G(run_scores_parts, 0, 0, a, D, st, ev0, ev1)
  }
  if (a.nl == 1) {
    const dim3 grid((a.n_tiles + 7) / 8, a.B);
    if (ev0 && ev1) hipExtLaunchKernelGGL(k_call_scores, grid, dim3(256), 0, st, ev0, ev1, 0, a, attn_step_tile_rows(D));
    else hipLaunchKernelGGL(k_call_scores, grid, dim3(256), 0, st, a, attn_step_tile_rows(D));
    return hipGetLastError();
  }
  const int tr = attn_step_tile_rows(D), threads = 64 * (a.nl < 16 ? a.nl : 16);
  if (ev0 && ev1) hipExtLaunchKernelGGL(k_step_scores, dim3(a.n_tiles, a.B), dim3(threads), 0, st, ev0, ev1, 0, a, tr);
  else hipLaunchKernelGGL(k_step_scores, dim3(a.n_tiles, a.B), dim3(threads), 0, st, a, tr);
  return hipGetLastError();
}

hipError_t launch_attn_finish(const AttnArgs& a, int D, int G, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  if (D == 128) { TKV_DISPATCH_G(run_finish, 128, KT_BF16, a, st, ev0, ev1) }
  if (D == 64) { TKV_DISPATCH_G(run_finish, 64, KT_BF16, a, st, ev0, ev1) }
  return hipErrorInvalidValue;
}

// ---- bandwidth probe: what a plain streaming read of `bytes` reaches with the attention kernel's launch shape ----
// One workgroup per compute unit, 512 lanes, 16-byte loads, four independent loads in flight per lane; nothing is
// written unless the data says so (it never does for the probe's buffer), so the traffic is the read alone.
__global__ __launch_bounds__(512) void k_probe_read(const u32x4* __restrict__ src, size_t n16, uint32_t* sink) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t acc = 0;
  for (; i + 3 * stride < n16; i += 4 * stride) {
    const u32x4 a = __builtin_nontemporal_load(src + i), b = __builtin_nontemporal_load(src + i + stride);
    const u32x4 c = __builtin_nontemporal_load(src + i + 2 * stride), d = __builtin_nontemporal_load(src + i + 3 * stride);
    acc ^= a.x ^ a.y ^ a.z ^ a.w ^ b.x ^ b.y ^ b.z ^ b.w ^ c.x ^ c.y ^ c.z ^ c.w ^ d.x ^ d.y ^ d.z ^ d.w;
  }
  for (; i < n16; i += stride) { const u32x4 a = __builtin_nontemporal_load(src + i); acc ^= a.x ^ a.y ^ a.z ^ a.w; }
  if (acc == 0x9E3779B9u) *sink = acc;
}
hipError_t launch_probe_read(const void* src, size_t bytes, int workgroups, uint32_t* sink, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  hipExtLaunchKernelGGL(k_probe_read, dim3(workgroups), dim3(512), 0, st, ev0, ev1, 0, (const u32x4*)src, bytes / 16, sink);
  return hipGetLastError();
}
#endif

}  // namespace tkv
