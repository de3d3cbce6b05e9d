// Decode attention over the packed cache (gfx950): out = softmax(scale * q K^^T) V^  (App. A of
// arXiv 2502.15075) with K^, V^ the group-wise reconstructions code*scale+zero (App. B), computed
// without ever materializing K^ or V^:
//
//   logit[t,h]  = sum_g  sK[t,g] * (sum_{d in g} q[h,d] cK[t,d])  +  zK[t,g] * (sum_{d in g} q[h,d])
//   out[h,d]    = ( sum_t (p[t,h] sV[t,g(d)]) cV[t,d]  +  sum_t p[t,h] zV[t,g(d)] ) / sum_t p[t,h]
//
// Both inner sums over codes are 16x16x32 f16 matrix instructions.  A b-bit code c placed in the
// low mantissa bits of a binary16 lane is the subnormal c * 2^-24 (or c * 2^(k-24) when left at bit
// k): the products with the query are exact and the sum is taken in a window of about 24 bits (see
// the note at k_slot_elem), so "unpacking" is one AND per two codes; the power-of-two position
// factors are divided out of the query operand once per wavefront.
//
// Work split: one workgroup (4 or 8 wavefronts) walks a contiguous range of 32-token steps of one
// (batch, kv head); its wavefronts interleave the steps and each carries all query heads of that kv
// head as matrix columns (column c = g*R + h: key group g, head h), so every cache byte is read
// once.  Each wavefront keeps a ring of steps in registers: after a step is computed its registers
// are refilled with the step one ring length ahead, so several steps of streaming loads are always
// in flight per wavefront.  Wavefronts merge through LDS, workgroups through a workspace of
// (max, sum, acc) records: a few are merged by the workgroup that finishes last, more by a small
// second kernel (merge_tag_for says how many).
//
// Variants of the same kernel (template parameters): unquantized rows as operands (bits = 16), key
// codes of 3 and 6 bits as a low and a high run with a query operand each, two column sets (8 heads
// with 32-channel groups), channel-wise key groups (Sec. 4 "Downstream Task
// Accuracy": the scale moves into a per-block query operand), paged planes (a page-table lookup per
// step), per-sequence lengths, the fused append of a decode step, Hadamard-rotated keys and values
// (Sec. 4 "Integration with Rotation-Based Methods").
#include "kvq_internal.h"
#include "kvq_quantizer.h"

#include <atomic>
#include <type_traits>

namespace kvq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// D += A(16x32) * B(32x16); operands travel as 4 dwords (8 x 16-bit), binary16 or bfloat16.
template <bool BF>
__device__ __forceinline__ float4v mma(u32x4 a, u32x4 b, float4v c) {
  if constexpr (BF) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

constexpr float kCodeUnit = 5.9604644775390625e-08f;  // 2^-24: value of a code's lowest mantissa bit
constexpr float kInvCodeUnit = 16777216.0f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kNegBig = -1.0e30f;


template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
// Sum over the 16/R lanes of a 16-lane row that share x's query head (lanes c, c+R, c+2R, ...).
template <int R>
__device__ __forceinline__ float sum_over_groups(float x) {
  if (R <= 8) x += dpp_f32<0x128>(x);   // row_ror:8
  if (R <= 4) x += dpp_f32<0x124>(x);   // row_ror:4
  if (R <= 2) x += dpp_f32<0x122>(x);   // row_ror:2
  if (R <= 1) x += dpp_f32<0x121>(x);   // row_ror:1
  return x;
}

// ---- two tiles side by side ------------------------------------------------------------------------------------------------
// Where a kv head's columns (heads times groups) fill no more than 8 of a tile's 16, the two 16-token tiles of a step lie side by
// side: lanes 0-7 of every row carry the columns for the step's first tile, lanes 8-15 the same columns for its second.  Both
// tiles are multiplied by the same query operand in all 16 columns, and each half keeps the product it is responsible for, so that a
// lane has 4 scores of its step instead of 8: half the scale and zero terms, exponentials, sums and weights (of 160 vector
// instructions a step of K4V2 40 fewer, and 4 of its 8 exponentials), and no sums over empty columns.  What it gives is issue time, which
// bounds every walk that does not bring the memory system to its rate.  8 and 4 scores, before the ring was cut to two
// steps, 4 query heads: 8 x 8 heads x 8192 tokens K4V2 15.8 and 15.0 us, channel-wise rotated keys 18.1 and 17.2, 16 x 8 x 16000
// K2V2 33.3 and 30.9, 16 sequences of 600 to 16001 tokens in pages 29.1 and 26.4, 32 x 8 x 32768 140.7 and 139.1.  The
// packed weights of the second tile come over by a rotation of the row (halves_swap) when the values are multiplied.  Column
// c & 7 of a half carries group (c & 7) % (8 / R) of head (c & 7) / (8 / R): groups next to each other, so that their sums are quad
// permutes, which stay inside the half.
template <int R>
__device__ __forceinline__ float sum_over_groups_half(float x) {
  if (R <= 4) x += dpp_f32<0xB1>(x);    // quad permutes: lane ^ 1, lane ^ 2
  if (R <= 2) x += dpp_f32<0x4E>(x);
  if (R <= 1) x += dpp_f32<0x141>(x);   // row_half_mirror: the other quad's total
  return x;
}
__device__ __forceinline__ uint32_t halves_swap(uint32_t x) {      // lane ^ 8's value (row_ror:8)
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x128, 0xF, 0xF, false);
}

// Sum (maximum) over the four 16-lane rows of a wavefront, in every lane: a swap of rows (of halves) leaves the two values to
// combine in the two registers.  Register permutes: through the LDS unit the same exchanges are a latency each in the chain
// that bounds a short launch.
__device__ __forceinline__ float rows_sum(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float rows_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// The same sum where channel-wise keys of BK bits rebuild their query operands, once per block in the main loop.  Keys of 1 and 2 bits, whose loop
// vector instructions bound, take it through the LDS permute unit, which saves 16 of 690 in a pair of steps; wider ones by
// register permutes.  In turn, register and LDS permutes (and before either was looked at), everything flushed: 32 x 8 x 8 heads x 32768 tokens
// K2V2 157.3 and 153.5 us (153.8), rotated keys 158.9 and 154.4 (155.7), K4V4 185.7 and 187.8 (188.5), K4V2 164.6 and 164.2; K1V4 2 % less, K2V8
// 8 x 8 x 32768 4 % less, K3V2 and K3V3 from 2 % less to 2 % more, K8V8 339.8 and 338.4.
template <int BK> __device__ __forceinline__ float kseq_rows_sum(float x) {
  if constexpr (BK > 2) return rows_sum(x);
  x += __shfl_xor(x, 16);
  x += __shfl_xor(x, 32);
  return x;
}
// Sum over groups of n = 4, 8 or 16 neighbouring lanes (uniform), in every lane.
__device__ __forceinline__ float lanes_sum(float x, int n) {
  x += dpp_f32<0xB1>(x);                // quad permutes: lane ^ 1, lane ^ 2
  x += dpp_f32<0x4E>(x);
  if (n > 4) x += dpp_f32<0x141>(x);    // row_half_mirror: the other quad's total
  if (n > 8) x += dpp_f32<0x140>(x);    // row_mirror: the other half's
  return x;
}

// ---- key codes: one lane holds 32 consecutive channels of one token (BK dwords) -------------
// (Channels 32j .. 32j+31 in the lanes of row quarter j.  A row of 16-bit patterns is 256 bytes, of which a lane would hold
// 4 neighbouring 16-byte pieces: every load instruction would touch every line of the tile and use a quarter of each.
// There a lane's pieces lie 64 bytes apart instead, so that the 4 lanes of a row read 64 bytes in one piece: element x (0..31)
// of row quarter j is channel 32 (x / 8) + 8 j + x % 8 (any assignment of channels to slots is as good as another for the
// matrix product, as long as the query operand follows it): the unquantized 8B layer at B=8, T=32768 takes 159 us = 6.74 TB/s where it took 201.  The same
// for the two pieces of 8-bit rows changes nothing (86.4 against 86.1 us for K8V8 there): lines are halves, not quarters.)
// Matrix step m (0..3) consumes 8 of them; slot i of that step is channel k_slot_elem(m,i) of the
// lane's 32, left at bit k of its 16-bit lane, i.e. read as code * 2^k * 2^-24, so the query operand of the slot is
// divided by k_slot_scale(i) = 2^k.
//
// Where the fields are left matters for accuracy.  A binary16 subnormal enters the matrix unit with the exponent
// 2^-14 whatever its leading zeros, and the unit keeps about 24 bits below the largest product exponent of a dot
// product: a code at bit 0 against an undivided query element loses everything below 2^-38 times that element (measured:
// up to 3e-4 code units per 32-term dot product, which the scale of a coarse key format on outlier-heavy keys turns
// into several 1e-3 of a logit), a code at bit k against the element divided by 2^k keeps 2^k times more.  The query
// operand in turn must stay a normal binary16 number, so k stays at or below 6.  Hence: 2-bit fields are moved to bits
// 4 and 6 (one more shift per matrix step), single bits to BASE..BASE+3; 4-bit fields stay at bits 0 and 4 and 8-bit
// fields at bit 0 (their scales are small and the error stays at the level of the value side's weight rounding; moving
// the 4-bit fields as well was measured: the same maximum error, 2.8 % more time for the headline format).
// BASE: lowest bit of the moved 1- and 2-bit fields (the high run of 3- and 6-bit codes is moved higher, its query
// operand carries the factor 2^LO and is still normal).
template <int BK> __device__ __forceinline__ constexpr int k_slot_elem(int m, int i) {
  const int v = i >> 1, x = i & 1;
  if (BK == 16) return 8 * m + i;
  if (BK == 1) return 4 * m + v + 16 * x;
  if (BK == 4) return 8 * m + v + 4 * x;
  if (BK == 8) return 8 * m + 4 * (v >> 1) + (v & 1) + 2 * x;
  return 16 * (m >> 1) + 4 * (m & 1) + v + 8 * x;  // BK == 2
}
template <int BK> constexpr int k_piece_stride() { return BK == 16 ? 64 : 16; }
// Bytes from the row's start to the first piece of the lanes of row quarter j.
template <int BK> __device__ __forceinline__ constexpr int k_lane_offset(int j) { return j * (BK == 16 ? 16 : 4 * BK); }
template <int BK> constexpr int k_default_base() { return BK == 2 ? 4 : BK == 1 ? 3 : 0; }
template <int BK, int BASE = k_default_base<BK>()> __device__ __forceinline__ constexpr float k_slot_scale(int i) {
  const int v = i >> 1;
  if (BK == 4) return (v & 1) ? 16.0f : 1.0f;
  if (BK == 8 || BK == 16) return 1.0f;
  if (BK == 1) return (float)(1 << (BASE + v));
  return (float)(1 << (BASE + 2 * (v & 1)));       // BK == 2
}
// One run of a key row's codes: B-bit fields left at BASE, whose query operand carries FACTOR.
template <int B, int BASE, int FACTOR> struct KRun { static constexpr int bits = B, base = BASE; static constexpr float factor = (float)FACTOR; };
// The query operand is staged by lanes that hold 8 neighbouring channels 8 o .. 8 o + 7 of a row, in operand order
// [row quarter j = o / 4][matrix step m][slot i].  For 4- and 8-bit fields these are the 8 slots of step o % 4; for 1- and
// 2-bit fields every other slot of two steps: channel e goes 16 (e / 4) + 4 (e % 4) bytes behind k_octet_offset.
template <int B> __device__ __forceinline__ constexpr int k_octet_offset(int o) {
  return (o >> 2) * 64 + (B == 2 ? ((o >> 1) & 1) * 32 + (o & 1) * 2 : (o & 1) * 32 + ((o >> 1) & 1) * 2);
}
template <int B, int BASE> __device__ __forceinline__ constexpr float k_octet_scale(int e) {
  return B == 8 || B == 16 ? 1.0f : k_slot_scale<B, BASE>(2 * (e & 3));
}
template <int B, int BASE> constexpr bool k_octet_matches() {
  for (int o = 0; o < 4; ++o)
    for (int e = 0; e < 8; ++e) {
      const int at = B == 4 ? o * 16 + 4 * (e & 3) + 2 * (e >> 2)
                   : B == 8 ? o * 16 + 8 * (e >> 2) + 4 * (e & 1) + 2 * ((e >> 1) & 1)
                            : k_octet_offset<B>(o) + 16 * (e >> 2) + 4 * (e & 3);
      const int m = at / 16, i = (at % 16) / 2;
      if (k_slot_elem<B>(m, i) != 8 * o + e || k_slot_scale<B, BASE>(i) != k_octet_scale<B, BASE>(e)) return false;
    }
  return true;
}
static_assert(k_octet_matches<1, k_default_base<1>()>() && k_octet_matches<2, k_default_base<2>()>() && k_octet_matches<4, 0>() &&
              k_octet_matches<8, 0>() && k_octet_matches<1, 5>() && k_octet_matches<2, 6>(), "staged query operands");
// The same factor as a function of the channel (the slot a channel lands in fixes it), default BASE.
template <int BK> __device__ __forceinline__ constexpr float k_chan_scale(int d) {
  return BK == 4 ? ((d & 1) ? 16.0f : 1.0f) : BK == 2 ? ((d & 1) ? 64.0f : 16.0f) : 1.0f;
}
template <int BK> constexpr bool k_chan_scale_matches() {
  for (int m = 0; m < 4; ++m)
    for (int i = 0; i < 8; ++i)
      if (k_chan_scale<BK>(k_slot_elem<BK>(m, i)) != k_slot_scale<BK>(i)) return false;
  return true;
}
static_assert(k_chan_scale_matches<2>() && k_chan_scale_matches<4>() && k_chan_scale_matches<8>(), "slot factors");
// (shift left by s, right for negative s; s is a compile-time value after unrolling)
__device__ __forceinline__ uint32_t shl_signed(uint32_t w, int s) { return s >= 0 ? w << s : w >> (-s); }
template <int BK, int BASE = k_default_base<BK>()> __device__ __forceinline__ u32x4 unpack_k(const uint32_t* w, int m) {
  u32x4 a;
  if constexpr (BK == 16) {
    a = u32x4{w[4 * m], w[4 * m + 1], w[4 * m + 2], w[4 * m + 3]};      // unquantized: the 16-bit patterns themselves
  } else if constexpr (BK == 4) {
    const uint32_t lo = w[m], hi = w[m] >> 8;
    a = u32x4{lo & 0x000F000Fu, lo & 0x00F000F0u, hi & 0x000F000Fu, hi & 0x00F000F0u};
  } else if constexpr (BK == 8) {
    const uint32_t w0 = w[2 * m], w1 = w[2 * m + 1];
    a = u32x4{w0 & 0x00FF00FFu, (w0 >> 8) & 0x00FF00FFu, w1 & 0x00FF00FFu, (w1 >> 8) & 0x00FF00FFu};
  } else if constexpr (BK == 1) {
    // bit 4m+v of each half (channels 4m+v and 16+4m+v) to bit BASE+v.  What a shift carries across the middle of the
    // word lands outside the masks: left shifts reach bit 16+BASE-1 at most, right shifts bit 16-(4m-BASE) at least.
    static_assert(BASE >= 0 && BASE <= 7, "single-bit fields stay below bit 11");
    const uint32_t ws = shl_signed(w[0], BASE - 4 * m);
    constexpr uint32_t k1 = 0x00010001u << BASE;
    a = u32x4{ws & k1, ws & (k1 << 1), ws & (k1 << 2), ws & (k1 << 3)};
  } else {
    // fields 0,1 of the byte (bits 0-3) and fields 2,3 (bits 4-7) both to bits BASE..BASE+3 (same remark on carries)
    static_assert(BASE >= 4 && BASE <= 7, "two-bit fields stay below bit 11");
    const int byte0 = 8 * (m & 1);
    const uint32_t wl = shl_signed(w[m >> 1], BASE - byte0), wh = shl_signed(w[m >> 1], BASE - 4 - byte0);
    constexpr uint32_t k2 = 0x00030003u << BASE;
    a = u32x4{wl & k2, wl & (k2 << 2), wh & k2, wh & (k2 << 2)};
  }
  return a;
}
// Key codes of 3 and 6 bits are a low run (2 / 4 bits, the first dwords of the lane's 32 channels) and a high run
// (1 / 2 bits, the rest): two operands, multiplied by the query separately (the high run's query operand carries the
// factor 2^LO).
template <int BK> constexpr int k_lo() { return code_lo_bits<BK>(); }
template <int BK> constexpr int k_hi() { return code_hi_bits<BK>(); }
template <int BK> constexpr int k_hi_base() { return BK == 3 ? 5 : 6; }   // high run: single bits from bit 5, pairs from bit 6

// ---- value codes: one lane holds, per 32-token step, 2*BV dwords (index = 4*piece + dword; 1-bit codes: one piece
// of two dwords, d-tile dt's 8 codes in nibble dt%4 of each half of dword dt/4) ----
// Register v (0..3) of d-tile dt's operand holds slots 2v, 2v+1 and is left at bit offset v_slot_shift(v)
// of its 16-bit lane, i.e. it reads as code * 2^shift * 2^-24; the softmax weight of those slots is
// divided by 2^shift instead (an exponent offset, free).
// Value codes of 3 and 6 bits are a block of low parts (2 / 4 bits) and a block of high parts (1 / 2 bits): two
// operands per d-tile; v_slot_shift is the low part's, and the high part's weights carry the factor v_hi_factor.
template <int BV> constexpr int v_lo() { return code_lo_bits<BV>(); }
template <int BV> constexpr int v_hi() { return code_hi_bits<BV>(); }
template <int B> __device__ __forceinline__ constexpr int field_slot_shift(int v) {
  return B == 1 ? v : B == 2 ? 2 * v : (B == 4 ? 4 * (v & 1) : 0);
}
template <int BV> __device__ __forceinline__ constexpr int v_slot_shift(int v) { return field_slot_shift<v_lo<BV>()>(v); }
// code = lo + 2^LO hi, and the two operands sit at different bit offsets of their 16-bit lanes
template <int BV> __device__ __forceinline__ constexpr float v_hi_factor(int v) {
  return (float)(1 << (v_lo<BV>() + field_slot_shift<v_lo<BV>()>(v))) / (float)(1 << field_slot_shift<(v_hi<BV>() ? v_hi<BV>() : 1)>(v));
}
// Softmax weights are carried times 2^p_shift and divided by 2^shift of their slot: the largest of them is 2^10 (binary16
// headroom for weight x value scale up to 64), so p_shift is 10 plus the smallest slot shift, where the high part's
// slots count with their shift minus LO (their weights carry 2^LO).  The scale of a 1-bit group is its whole range:
// two bits more headroom (scale up to 255).  Larger scales: see weight_headroom.
template <int BV> constexpr float p_shift() {
  int m = field_slot_shift<v_lo<BV>()>(0);
  if (v_hi<BV>()) {
    const int h = field_slot_shift<(v_hi<BV>() ? v_hi<BV>() : 1)>(0) - v_lo<BV>();
    m = h < m ? h : m;
  }
  return (float)(10 + m - (BV == 1 ? 2 : 0));
}
template <int BV> __device__ __forceinline__ u32x4 unpack_v(const uint32_t* w, int dt) {
  u32x4 a;
  if (BV == 16) {
    a = u32x4{w[4 * dt], w[4 * dt + 1], w[4 * dt + 2], w[4 * dt + 3]};
  } else if (BV == 1) {
    const uint32_t ws = w[dt >> 2] >> (4 * (dt & 3));
    a = u32x4{ws & 0x00010001u, ws & 0x00020002u, ws & 0x00040004u, ws & 0x00080008u};
  } else if (BV == 2) {
    const uint32_t ws = w[dt >> 1] >> (8 * (dt & 1));
    a = u32x4{ws & 0x00030003u, ws & 0x000C000Cu, ws & 0x00300030u, ws & 0x00C000C0u};
  } else if (BV == 4) {
    const uint32_t lo = w[dt], hi = lo >> 8;
    a = u32x4{lo & 0x000F000Fu, lo & 0x00F000F0u, hi & 0x000F000Fu, hi & 0x00F000F0u};
  } else {
    const uint32_t w0 = w[2 * dt], w1 = w[2 * dt + 1];
    a = u32x4{w0 & 0x00FF00FFu, (w0 >> 8) & 0x00FF00FFu, w1 & 0x00FF00FFu, (w1 >> 8) & 0x00FF00FFu};
  }
  return a;
}

#ifndef KVQ_STAGES
#define KVQ_STAGES 2           // 32-token steps resident or in flight per wavefront (register ring)
#endif
#ifndef KVQ_WAVES_PER_SIMD
#define KVQ_WAVES_PER_SIMD 2   // what the register allocation leaves room for at least, and the plan counts on
#endif

// Ring depth per instantiation: two steps, one where the registers of a step (2 b_K + 2 b_V + 4 per lane) leave no room for a second.
// Eight wavefronts with one step each in flight, 28 KB of K4V2 per unit, keep the memory system busy; a deeper ring only makes the
// first fill, which every wavefront asks for at once, and the code longer.  With 6, 4, 3, 2 and 1 steps, K4V2: 8 x 8 heads x 8192 tokens
// 16.7, 15.2, 14.4, 14.1 and 15.4 us, 8 heads x 131071 26.9, 25.4, 24.4, 24.1 and 26.3, 32 x 8 x 8 heads x 32768 143.3, 141.7, 142.0, 140.6 and
// 164.1; K4V4 with 3, 2 and 1: 8 x 8 x 8192 17.1, 16.7 and 17.1, 40 x 8 x 3000 30.8, 29.6 and 33.4; K2V2 with 4, 3, 2: 13.4, 12.6, 12.5.
// Three where the columns fill a tile and a row has up to 5 bits (one step of the walk then takes as long as the data of the next to come, and
// walks of three steps are common): 8 query heads, with 4, 2 and 3, K2V2 2 x 8 heads x 6000 tokens 10.1, 10.5 and 10.1, x 8 x 8192 15.7, 15.1
// and 15.1; K4V1 in 32-channel value groups 5 x 8 x 6049 13.5, 13.8 and 13.3; K3V2 8 x 8 x 2000 10.4, 10.6 and 10.5.
template <int BK, int BV, int NCK = 1, int NCV = 1, bool ROTV = false, bool HALF = false>
constexpr int ring_stages() {
  if (HALF) return KVQ_STAGES;
  constexpr int regs = 2 * BK + 2 * BV + 4;
  constexpr int base = regs <= 16 ? 4 : regs <= 20 ? 3 : 2;
  constexpr int less = (NCK == 2 ? 2 : 0) + (NCV == 2 ? 1 : 0)    // a second column set costs registers (query operand,
                       + (code_hi_bits<BK>() ? 1 : 0)              // scale/zero entries, weights), so does a high run
                       + (code_hi_bits<BV>() ? 1 : 0)              // of keys or a high part of values (its weights)
                       + (ROTV ? 1 : 0)                            // (rotated values: the unrounded weights stay live)
                       + (BK == 2 && regs >= 16 ? 1 : 0);         // (moved 2-bit fields: two shifted copies of a word live)
  constexpr int most = regs <= 14 ? KVQ_STAGES + 1 : KVQ_STAGES;
  return base - less >= most ? most : base - less >= 1 ? base - less : 1;
}

// Everything one lane loads for one 32-token step (two 16-token tiles).
template <int BK, int BV>
struct StepRegs {
  __attribute__((aligned(16))) uint32_t kc[2][BK];            // tile x4: row 16*x4 + c, this lane's 32 channels
  __attribute__((aligned(16))) uint32_t vc[2 * BV];           // value codes: piece k, dword m at [4k + m]
  u32x4 meta;                    // 16 bytes of the step's scale/zero bytes, in plane order (lane l < 8 (ng_k + ng_v) holds
                                 // bytes 16 l ..); redistributed through LDS when the step is computed
};

struct LaneCtx {
  const uint8_t* kc; const uint8_t* vc;   // (b,h) stream bases of the code planes (wave-uniform)
  const uint8_t* meta_base;               // this lane's scale/zero plane: key plane for lanes < 8 ng_k, else value plane
  uint32_t meta_mul, meta_off;            // bytes of that plane per 32-token step; this lane's offset inside them
  uint32_t meta_step_mask;                // ~1 for the key lanes of channel-wise keys (one entry set per two steps)
  uint32_t kc_off, vc_off;                // this lane's byte offsets inside one step of the code planes
  uint32_t km_rd, vm_rd;                  // byte offsets of this lane's key / value scale-zero entries (tile 0) in the
                                          // wavefront's LDS copy of a step's scale/zero bytes
  uint8_t* meta_lds;                      // that LDS copy (1 KB per wavefront)
  int lane, c, j, gk, gv, ngk, ngv;
  static constexpr bool kRotV = false;
};
// Kernels for caches whose values are stored rotated (the output goes through R_v^T) mark their context so.
struct LaneCtxRotV : LaneCtx { static constexpr bool kRotV = true; };

// Addresses formed by integer arithmetic name global memory explicitly: a pointer of unknown address space becomes a flat
// access, which may return out of order with everything else, so that the compiler drains ALL loads in flight at the
// next wait (the ring's first fill among them).
template <typename T> __device__ __forceinline__ T load_global(uintptr_t p) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(p);
}
template <typename T> __device__ __forceinline__ void store_global(uintptr_t p, T v) {
  *reinterpret_cast<__attribute__((address_space(1))) T*>(p) = v;
}

// Cache bytes are read exactly once per decode step: streaming (non-temporal) loads.
__device__ __forceinline__ u32x4 ld16(const uint8_t* p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
}

// WIDE (paged planes): `step` counts 32-token steps in plane order from the plane base, so the uniform part of the
// address is formed in 64 bits; otherwise it counts inside the (b,h) stream that the bases point to.
// N consecutive dwords of a key tile (4 N bytes per lane: the lane's 32 channels), non-temporal; the address is a
// multiple of 4 N bytes only when N is a power of two (3- and 6-bit rows), so the vector types carry that alignment.
// STRIDE: bytes between a lane's 16-byte pieces (pieces of 16 bytes and more)
template <int N, int STRIDE = 16> __device__ __forceinline__ void load_dwords(uint32_t* dst, const uint8_t* p) {
  typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(8)));
  typedef uint32_t v3 __attribute__((ext_vector_type(3), aligned(4)));
  typedef uint32_t v4a8 __attribute__((ext_vector_type(4), aligned(8)));
  if constexpr (N == 1) {
    dst[0] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
  } else if constexpr (N == 2) {
    const v2 v = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
    dst[0] = v.x; dst[1] = v.y;
  } else if constexpr (N == 3) {
    const v3 v = __builtin_nontemporal_load(reinterpret_cast<const v3*>(p));
    dst[0] = v.x; dst[1] = v.y; dst[2] = v.z;
  } else if constexpr (N == 6) {
    const v4a8 v = __builtin_nontemporal_load(reinterpret_cast<const v4a8*>(p));
    dst[0] = v.x; dst[1] = v.y; dst[2] = v.z; dst[3] = v.w;
    load_dwords<2>(dst + 4, p + 16);
  } else {
    static_assert(N % 4 == 0, "key tile piece");
#pragma unroll
    for (int k = 0; k < N / 4; ++k) {
      const u32x4 v = ld16(p + STRIDE * k);
      *reinterpret_cast<u32x4*>(dst + 4 * k) = v;
    }
  }
}

// lane_mask: ~0, or 0 for a refill past the wavefront's last step, which still issues its loads (every lane then reads
// the first 16 bytes of each part of the step it is given: one cache line per load, the data is never used).  A load
// that may or may not be issued sits behind a branch, and with a branch between the loads the compiler can no longer
// count how many newer loads follow a ring slot's: it then drains the ring before every use.
template <int BK, int BV, bool WIDE = false>
__device__ __forceinline__ void load_step(StepRegs<BK, BV>& r, const LaneCtx& L, int64_t step, uint32_t lane_mask = ~0u) {
  // uniform 64-bit base + 32-bit offset (a (b,h) stream of any plane is below 4 GiB)
  const uint8_t* kbase = WIDE ? L.kc + step * (512 * BK) : L.kc;
  const uint8_t* vbase = WIDE ? L.vc + step * (512 * BV) : L.vc;
  const uint8_t* mbase = WIDE ? L.meta_base + (step & (int64_t)(int32_t)L.meta_step_mask) * L.meta_mul : L.meta_base;
  const uint32_t ko = (WIDE ? 0u : (uint32_t)step * (512 * BK)) + (L.kc_off & lane_mask);
#pragma unroll
  for (int x4 = 0; x4 < 2; ++x4) load_dwords<BK, k_piece_stride<BK>()>(r.kc[x4], kbase + (ko + x4 * (256 * BK)));
  // (every lane loads, for the same reason: lanes beyond the scale/zero bytes repeat the last 16 of them)
  if constexpr (BK != 16 || BV != 16)
    r.meta = ld16(mbase + ((WIDE ? 0u : ((uint32_t)step & L.meta_step_mask) * L.meta_mul) + (L.meta_off & lane_mask)));
  constexpr int VLO = v_lo<BV>(), VHI = v_hi<BV>();
  const uint32_t vstep = WIDE ? 0u : (uint32_t)step * (512 * BV);
  const uint32_t vo = vstep + (L.vc_off & lane_mask);
  if constexpr (BV == 1) load_dwords<2>(r.vc, vbase + vo);
#pragma unroll
  for (int k = 0; k < VLO / 2; ++k) {
    const u32x4 v = ld16(vbase + (vo + k * 1024));
    *reinterpret_cast<u32x4*>(r.vc + 4 * k) = v;
  }
  // the block of high parts follows the block of low parts: 8 bytes per lane (single bits) or 16 (pairs)
  if constexpr (VHI == 1) load_dwords<2>(r.vc + 2 * VLO, vbase + (vstep + 512 * VLO + ((L.vc_off >> 1) & lane_mask)));
  if constexpr (VHI == 2) load_dwords<4>(r.vc + 2 * VLO, vbase + (vstep + 512 * VLO + (L.vc_off & lane_mask)));
}

__device__ __forceinline__ float meta_scale(uint32_t m) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(m & 0xFFFFu)); }
__device__ __forceinline__ float meta_zero(uint32_t m) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(m >> 16)); }

template <int NCV, bool HALF = false>
struct WaveState {
  static constexpr int kClasses = HALF ? 2 : 4;  // register classes of a lane's scores (HALF: v or v + 2, by the lane's tile)
  float4v acc[8];       // out^T tile dt: rows d = 16*dt + 4*j + r, column c
  float m;              // running max of this lane's head, in log2 units
  float noff[kClasses]; // p_shift - m - v_slot_shift(v): exponent offset of the slots in operand register v
  float l[kClasses];    // per register class v: this lane's share of sum_t p * 2^(p_shift - shift(v))
  float zacc[NCV][kClasses];   // same, weighted by zV[t, g] for this lane's value group of each column set
  float headroom;       // the running maximum is kept this far (in log2 units) above the largest logit seen, which holds
                        // every weight below 2^-headroom of its usual size (see weight_headroom); wave-uniform
};

// The softmax weights go into the matrix unit as binary16 products p * 2^p_shift * scale_V, and the largest of them
// (p = 1 at the running maximum) stays finite only for value scales below 2^(16 - p_shift) = 64 (256 for 1-bit values),
// i.e. for groups whose range is below 64 (2^b - 1) -- while inputs may be as large as binary16 goes.  The append
// kernels therefore keep, per (batch, kv head), the largest exponent field of any value scale they have stored
// (kvq_cache.v_scale_exp), and an attention launch over a stream that holds a scale of 64 or more holds ALL its
// weights down: the running maximum stays (that exponent - 5) above the logits, which divides every weight and every
// sum by that power of two (the final division by the sum of weights takes it out again).  What it costs is resolution
// of the smallest weights, which such a stream can spare: they multiply values of the same large scale.  Nothing of
// this is in the loop: the offset rides in the multiply-add that turns a logit into log2 units.
template <int BV> __device__ __forceinline__ float weight_headroom(int scale_exp_field) {
  const int need = scale_exp_field - 15 - (BV == 1 ? 7 : 5);   // scales below 2^6 (1-bit values: 2^8) need nothing
  return (float)(need < 0 ? 0 : need > 16 ? 16 : need);
}

// binary16 product of a binary32 weight and the binary16 held in the low half of `meta`, written to the
// low / high half of `dst` (one rounding: the compiler turns the fused multiply-add with a converted operand and the
// conversion of its result into one v_fma_mixlo/mixhi_f16).  Written in C and not as inline assembly on purpose: the
// weight comes straight from v_exp_f32, and the result of a transcendental instruction may not be read by the next
// vector instruction; the compiler keeps that distance for the instructions it emits itself, not for assembly text.
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void mix_lo(uint32_t& dst, float p, uint32_t meta) {
  const half2v r = {(_Float16)fmaf(p, meta_scale(meta), 0.0f), (_Float16)0.0f};
  dst = __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ void mix_hi(uint32_t& dst, float p, uint32_t meta) {
  half2v r = __builtin_bit_cast(half2v, dst);
  r.y = (_Float16)fmaf(p, meta_scale(meta), 0.0f);
  dst = __builtin_bit_cast(uint32_t, r);
}

// Round-to-nearest-even bfloat16 pattern of a finite binary32.
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// ---- channel-wise keys (one scale/zero per channel and 64-token block) --------------------------------------------
// The scale of channel d cannot leave the contraction over d, so it is folded into the query: per block the operand
// q~[h,d] = q[h,d] * sK[blk,d] is rebuilt, as a high and a low binary16 part (the product of two 11-bit numbers has
// 22 bits; the low part carries the rest down to an absolute 2^-25, far below what the scores resolve).  The two parts
// are two matrix columns of the same head (column group 0 the high part, group 1 the low part: at most 8 heads fill
// 16 columns), so one matrix instruction multiplies the codes by both and the sum over column groups that the
// token-wise kernel uses for its key groups adds them.  The zero points enter as one constant per head and block,
// sum_d q[h,d] zK[blk,d].  logit[t,h] = sum_d q~[h,d] cK[t,d] + that constant.
struct KSeqState {
  u32x4 qop[4];            // query operand of the current block: this lane's part (high or low) of its head
  float zq_u;              // zero-point term of the current block, in code units (lanes of the high part; else 0)
};
struct KSeqState2 : KSeqState {
  u32x4 qoph[4];           // the same for the high run of 3- and 6-bit key codes (carries the factor 2^LO)
};
struct NoKSeq {};
// 2-, 4- and 8-bit keys: the staged query row is already divided by the position factor of each channel's code
// (k_chan_scale).  1-, 3- and 6-bit keys: the row is staged as it is and the factors of each run's slots are applied
// when the operands are built.
template <int BK> constexpr bool kseq_prescaled() { return BK == 2 || BK == 4 || BK == 8; }

// Rebuild the block's query operand from the staged query row and the block's 128 scale/zero entries (first 512 bytes
// of the wavefront's LDS copy of the step's scale/zero bytes).
// qrow: the head's query in binary32, channel d divided by k_chan_scale(d) (LDS; an all-zero row for a lane whose
// column carries nothing on the key side).  low_part: 1.0f in the lanes of the low part, 0.0f in those of the high part.
// The high part is the product rounded toward zero, h = rtz16(v); every lane forms v - low_part * h and converts
// again: v's own high part where low_part is 0, the exact rest where it is 1 — the same instructions in both.
template <int BK>
__device__ __forceinline__ void kseq_rebuild(KSeqState& ks, const LaneCtx& L, const float* qrow, float low_part) {
  constexpr int NC = BK == 8 ? 1 : 2;                        // classes of channels by k_chan_scale (even / odd)
  typedef __fp16 half2v __attribute__((ext_vector_type(2)));
  float zc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) zc[c] = 0.f;
  const float nlow = -low_part;
#pragma unroll
  for (int half32 = 0; half32 < 2; ++half32) {     // 16 channels at a time: matrix steps 2*half32 and 2*half32 + 1
    float w[16];
#pragma unroll
    for (int quad = 0; quad < 4; ++quad) {
      const float4v qf = *reinterpret_cast<const float4v*>(qrow + 32 * L.j + 16 * half32 + 4 * quad);
      const u32x4 mv = *reinterpret_cast<const u32x4*>(L.meta_lds + 128 * L.j + 64 * half32 + 16 * quad);
      const uint32_t mw[4] = {mv.x, mv.y, mv.z, mv.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[4 * quad + e] = fmaf(qf[e], meta_scale(mw[e]), 0.0f);
        zc[e % NC] = fmaf(qf[e], meta_zero(mw[e]), zc[e % NC]);
      }
    }
#pragma unroll
    for (int mm = 0; mm < 2; ++mm) {
      const int m = 2 * half32 + mm;
      uint32_t op[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float a = w[k_slot_elem<BK>(m, 2 * v) - 16 * half32], b = w[k_slot_elem<BK>(m, 2 * v + 1) - 16 * half32];
        const half2v h = __builtin_amdgcn_cvt_pkrtz(a, b);
        const float xa = fmaf((float)h.x, nlow, a), xb = fmaf((float)h.y, nlow, b);
        op[v] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(xa, xb));
      }
      ks.qop[m] = u32x4{op[0], op[1], op[2], op[3]};
    }
  }
  float zq = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c) zq = fmaf(zc[c], k_chan_scale<BK>(c), zq);
  zq = kseq_rows_sum<BK>(zq);
  ks.zq_u = zq * (kCodeUnit - kCodeUnit * low_part);          // (only the high part's column adds the constant)
}

// The same for 1-, 3- and 6-bit keys: all 32 products q[d] sK[d] of the lane first (a single-bit run takes a matrix
// step's channels from both halves of the 32), then one operand set per run, each slot divided by the power of two at
// which the run's codes are left in their 16-bit lanes, the high run's times 2^LO.
template <int BK, typename KS>
__device__ __forceinline__ void kseq_rebuild_runs(KS& ks, const LaneCtx& L, const float* qrow, float low_part) {
  constexpr int KLO = k_lo<BK>(), KHI = k_hi<BK>();
  typedef __fp16 half2v __attribute__((ext_vector_type(2)));
  const float nlow = -low_part;
  float w[32];
  float zq = 0.f;
#pragma unroll
  for (int quad = 0; quad < 8; ++quad) {
    const float4v qf = *reinterpret_cast<const float4v*>(qrow + 32 * L.j + 4 * quad);
    const u32x4 mv = *reinterpret_cast<const u32x4*>(L.meta_lds + 128 * L.j + 16 * quad);
    const uint32_t mw[4] = {mv.x, mv.y, mv.z, mv.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      w[4 * quad + e] = fmaf(qf[e], meta_scale(mw[e]), 0.0f);
      zq = fmaf(qf[e], meta_zero(mw[e]), zq);
    }
  }
  auto part16 = [&](float a, float b) -> uint32_t {          // this lane's part (high or low) of the pair, see above
    const half2v h = __builtin_amdgcn_cvt_pkrtz(a, b);
    const float xa = fmaf((float)h.x, nlow, a), xb = fmaf((float)h.y, nlow, b);
    return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(xa, xb));
  };
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    uint32_t op[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float f = 1.0f / k_slot_scale<KLO>(2 * v);
      op[v] = part16(w[k_slot_elem<KLO>(m, 2 * v)] * f, w[k_slot_elem<KLO>(m, 2 * v + 1)] * f);
    }
    ks.qop[m] = u32x4{op[0], op[1], op[2], op[3]};
    if constexpr (KHI != 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float f = (float)(1 << KLO) / k_slot_scale<KHI, k_hi_base<BK>()>(2 * v);
        op[v] = part16(w[k_slot_elem<KHI>(m, 2 * v)] * f, w[k_slot_elem<KHI>(m, 2 * v + 1)] * f);
      }
      ks.qoph[m] = u32x4{op[0], op[1], op[2], op[3]};
    }
  }
  zq = kseq_rows_sum<BK>(zq);
  ks.zq_u = zq * (kCodeUnit - kCodeUnit * low_part);
}

// One 32-token step.  MASKED: tokens at or beyond seq_len get weight 0 (garbage may sit there).
// BK == BV == 16 is the unquantized cache: no scale/zero, operands are the stored patterns (BF: bfloat16).
// NCK / NCV: column sets.  Columns are (group, head) pairs; when R * (groups) exceeds the 16 columns of a matrix tile
// (8 heads with 32-channel groups) the groups are spread over two column sets: set cs carries group grp + cs*(16/R).
// KS: KSeqState for channel-wise keys (then NEWBLK marks the first step of a 64-token block: the query operands are
// rebuilt from that block's scale/zero entries), NoKSeq otherwise.
// HALF: the two tiles side by side (quantized tensors, one column set).
template <int BK, int BV, int R, bool BF, int NCK, int NCV, bool MASKED, bool NEWBLK = false, bool HALF = false, typename KS = NoKSeq,
          typename LC = LaneCtx>
__device__ __forceinline__ void compute_step(const StepRegs<BK, BV>& r, const u32x4 (&qb)[NCK][4],
                                             const u32x4 (&qbh)[NCK][4], const float (&qsum_u)[NCK],
                                             float kappa, WaveState<NCV, HALF>& st, const LC& L, int step, int seq_len,
                                             KS& ks, const float* qrow = nullptr, float kseq_low = 0.f,
                                             bool rebuild = true) {
  // a tensor of bits = 16 is stored as its 16-bit patterns (BF: bfloat16) and multiplied as it is, no scale/zero
  constexpr bool RAWK = BK == 16, RAWV = BV == 16;
  constexpr bool BFK = RAWK && BF, BFV = RAWV && BF;
  constexpr int KLO = k_lo<BK>(), KHI = k_hi<BK>();   // qbh: the query operand of the high run (3- and 6-bit keys)
  constexpr bool KSEQ = !__is_same(KS, NoKSeq);
  static_assert(!HALF || (!RAWK && !RAWV && NCK == 1 && NCV == 1), "two tiles side by side: quantized tensors, one column set");
  constexpr int NS = HALF ? 4 : 8;               // scores of this lane: slot i of tile i / 4 (HALF: of its half's tile)
  const bool upper = HALF && (L.c & 8);
  constexpr int kSetStride = (16 / R) * 64;      // bytes between the scale/zero entries of a lane's groups in two sets
  uint32_t kmeta[NCK][NS], vmeta[NCV][NS];
  if constexpr (!RAWK || !RAWV) {
    // scale/zero bytes: plane order -> LDS -> the entries this lane needs (tokens 4j..4j+3 of both tiles, own groups)
    *reinterpret_cast<u32x4*>(L.meta_lds + L.lane * 16) = r.meta;     // (lanes beyond the bytes fill slots nobody reads)
    if constexpr (KSEQ && NEWBLK) {
      if (rebuild) {                             // (uniform; false only in the second step of a group of 64 or 128 tokens)
        if constexpr (kseq_prescaled<BK>()) kseq_rebuild<BK>(ks, L, qrow, kseq_low);
        else kseq_rebuild_runs<BK>(ks, L, qrow, kseq_low);
      }
    }
#pragma unroll
    for (int x4 = 0; x4 < (HALF ? 1 : 2); ++x4) {
#pragma unroll
      for (int cs = 0; cs < NCK; ++cs) {
        if constexpr (KSEQ || RAWK) continue;
        const u32x4 a = *reinterpret_cast<const u32x4*>(L.meta_lds + L.km_rd + cs * kSetStride + x4 * (64 * L.ngk));
        kmeta[cs][4 * x4 + 0] = a.x; kmeta[cs][4 * x4 + 1] = a.y; kmeta[cs][4 * x4 + 2] = a.z; kmeta[cs][4 * x4 + 3] = a.w;
      }
#pragma unroll
      for (int cs = 0; cs < NCV; ++cs) {
        if constexpr (RAWV) continue;
        const u32x4 b = *reinterpret_cast<const u32x4*>(L.meta_lds + L.vm_rd + cs * kSetStride + x4 * (64 * L.ngv));
        vmeta[cs][4 * x4 + 0] = b.x; vmeta[cs][4 * x4 + 1] = b.y; vmeta[cs][4 * x4 + 2] = b.z; vmeta[cs][4 * x4 + 3] = b.w;
      }
    }
  }

  // ---- scores: slot i = token 16*(i/4) + 4*j + i%4 of this step (HALF: token 16*tile + 4*j + i)
  float s[NS];
  {
    float part[NS];
    auto own = [&](const float4v& d0, const float4v& d1, int i) { return HALF ? (upper ? d1[i & 3] : d0[i & 3]) : i < 4 ? d0[i & 3] : d1[i & 3]; };
    if constexpr (KSEQ) {
      float4v d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < 4; ++m) {                // two independent accumulation chains (the two 16-token tiles)
        d0 = mma<BF>(unpack_k<KLO>(r.kc[0], m), ks.qop[m], d0);
        d1 = mma<BF>(unpack_k<KLO>(r.kc[1], m), ks.qop[m], d1);
        if constexpr (KHI != 0) {
          d0 = mma<BF>(unpack_k<KHI, k_hi_base<BK>()>(r.kc[0] + KLO, m), ks.qoph[m], d0);
          d1 = mma<BF>(unpack_k<KHI, k_hi_base<BK>()>(r.kc[1] + KLO, m), ks.qoph[m], d1);
        }
      }
#pragma unroll
      for (int i = 0; i < NS; ++i) part[i] = own(d0, d1, i) + ks.zq_u;
    }
#pragma unroll
    for (int cs = 0; cs < NCK; ++cs) {
      if constexpr (KSEQ) continue;
      float4v d0 = {0.f, 0.f, 0.f, 0.f}, d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int m = 0; m < 4; ++m) {                // two independent accumulation chains
        d0 = mma<BFK>(unpack_k<KLO>(r.kc[0], m), qb[cs][m], d0);
        d1 = mma<BFK>(unpack_k<KLO>(r.kc[1], m), qb[cs][m], d1);
        if constexpr (KHI != 0) {
          d0 = mma<BFK>(unpack_k<KHI, k_hi_base<BK>()>(r.kc[0] + KLO, m), qbh[cs][m], d0);
          d1 = mma<BFK>(unpack_k<KHI, k_hi_base<BK>()>(r.kc[1] + KLO, m), qbh[cs][m], d1);
        }
      }
#pragma unroll
      for (int i = 0; i < NS; ++i) {
        const float d = own(d0, d1, i);
        float pt = d;
        if constexpr (!RAWK) pt = fmaf(d, meta_scale(kmeta[cs][i]), fmaf(meta_zero(kmeta[cs][i]), qsum_u[cs], 0.0f));
        part[i] = cs == 0 ? pt : part[i] + pt;
      }
    }
#pragma unroll
    for (int i = 0; i < NS; ++i) s[i] = HALF ? sum_over_groups_half<R>(part[i]) : sum_over_groups<R>(part[i]);
  }
  bool valid[NS];
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    valid[i] = !MASKED || (step * 32 + 16 * (HALF ? (L.c >> 3) : i >> 2) + 4 * L.j + (i & 3) < seq_len);
    if (MASKED && !valid[i]) s[i] = kNegBig;
  }
  // ---- running max (kept st.headroom above the logits): only when some lane sees a larger logit than its current max
  float lmax = fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
  if constexpr (!HALF) lmax = fmaxf(lmax, fmaxf(fmaxf(s[4], s[5]), fmaxf(s[6], s[7])));
  float lx = fmaf(lmax, kappa, st.headroom);
  if (__any(lx > st.m)) {
    if constexpr (HALF) lx = fmaxf(lx, __uint_as_float(halves_swap(__float_as_uint(lx))));      // (both halves of a head share its maximum)
    const float m_new = fmaxf(st.m, rows_max(lx));
    const float f = __builtin_amdgcn_exp2f(st.m - m_new);
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) st.acc[dt] *= f;
#pragma unroll
    for (int v = 0; v < st.kClasses; ++v) {
      st.l[v] *= f;
#pragma unroll
      for (int cs = 0; cs < NCV; ++cs) st.zacc[cs][v] *= f;
      st.noff[v] = p_shift<BV>() - (float)(upper ? v_slot_shift<BV>(v + 2) : v_slot_shift<BV>(v)) - m_new;
    }
    st.m = m_new;
  }
  // ---- softmax weights; quantized values: their binary16 products with the value scale, and the value-zero term
  constexpr int VLO = v_lo<BV>(), VHI = v_hi<BV>();
  uint32_t pw[NCV][4], pl[4];                    // pl: low-order bfloat16 part of the weights (bfloat16 cache only)
  uint32_t pwh[NCV][4];                          // weights of the high parts of 3- and 6-bit value codes
  constexpr bool ROTV = !RAWK && !RAWV && !KSEQ && LC::kRotV;   // (rotation is not combined with channel-wise keys)
  float pv[ROTV ? NS : 1];
  // (the high part's factor of class v, and what it is divided by again: the lane's own class)
  auto hi_factor = [&](int v) { return upper ? v_hi_factor<BV>(v + 2) : v_hi_factor<BV>(v); };
#pragma unroll
  for (int i = 0; i < NS; ++i) {
    const int v = i >> 1;
    float p = __builtin_amdgcn_exp2f(fmaf(s[i], kappa, st.noff[v]));
    if (MASKED && !valid[i]) p = 0.f;
    if constexpr (ROTV) pv[i] = p;
    st.l[v] += p;
    if constexpr (!RAWV) {
#pragma unroll
      for (int cs = 0; cs < NCV; ++cs) {
        uint32_t vm = vmeta[cs][i];
        if (MASKED && !valid[i]) vm = 0u;
        st.zacc[cs][v] = fmaf(p, meta_zero(vm), st.zacc[cs][v]);
        if (i & 1) mix_hi(pw[cs][v], p, vm); else mix_lo(pw[cs][v], p, vm);
        if constexpr (VHI != 0) {
          const float ph = p * hi_factor(v);
          if (i & 1) mix_hi(pwh[cs][v], ph, vm); else mix_lo(pwh[cs][v], ph, vm);
        }
      }
    } else if constexpr (!BF) {
      if (i & 1) mix_hi(pw[0][v], p, 0x3C00u); else mix_lo(pw[0][v], p, 0x3C00u);    // times binary16 1.0
    } else {
      // bfloat16 keeps 8 bits: carry the weight as two bfloat16 terms (16 bits) and multiply the values by both
      const uint32_t hi = bf16_rne(p);
      const uint32_t lo = bf16_rne(p - __uint_as_float(hi << 16));
      if (i & 1) { pw[0][v] |= hi << 16; pl[v] |= lo << 16; } else { pw[0][v] = hi; pl[v] = lo; }
    }
  }
  if constexpr (ROTV) {
    // Rotated values: the rounding error of a token's binary16 weight multiplies all of its group's codes alike, and
    // R_v^T gathers what is common to the channels into single output channels (times sqrt(D) for one group per row),
    // while the zero-point term beside it is summed with the unrounded weight.  What the rounding took from the weight
    // is therefore given back at the middle of the code range, through the zero-point sum: the error left is the
    // rounding error times the codes' distance from the middle, which has no common part to gather.
    constexpr float kMidLo = 0.5f * (float)((1 << VLO) - 1);
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      const int v = i >> 1;
#pragma unroll
      for (int cs = 0; cs < NCV; ++cs) {
        uint32_t vm = vmeta[cs][i];
        if (MASKED && !valid[i]) vm = 0u;
        const float back = (float)__builtin_bit_cast(_Float16, (uint16_t)((i & 1) ? pw[cs][v] >> 16 : pw[cs][v] & 0xFFFFu));
        st.zacc[cs][v] = fmaf(kMidLo, fmaf(pv[i], meta_scale(vm), -back), st.zacc[cs][v]);
        if constexpr (VHI != 0) {
          constexpr float kMidHi = 0.5f * (float)((1 << VHI) - 1) * (float)(1 << VLO);
          const float f = hi_factor(v);
          const float backh = (float)__builtin_bit_cast(_Float16, (uint16_t)((i & 1) ? pwh[cs][v] >> 16 : pwh[cs][v] & 0xFFFFu));
          st.zacc[cs][v] = fmaf(upper ? kMidHi / v_hi_factor<BV>(v + 2) : kMidHi / v_hi_factor<BV>(v), fmaf(pv[i] * f, meta_scale(vm), -backh), st.zacc[cs][v]);
        }
      }
    }
  }
  if constexpr (HALF) {                          // the other tile's weights, of the same head and value group (lanes 0-7 need them)
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      pw[0][v + 2] = halves_swap(pw[0][v]);
      if constexpr (VHI != 0) pwh[0][v + 2] = halves_swap(pwh[0][v]);
    }
  }
  // (Nothing is scheduled across this point.  The matrix instructions below cannot start before the weights are
  // complete anyway; left free, the scheduler pulls the unpacking of the value codes up into the softmax arithmetic,
  // which costs the kernel a dozen registers it does not have: with the fence no instance of the token-wise kernels
  // spills, without it most do.)
  if constexpr (!KSEQ) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) {
    constexpr int kDtPerSet = 8 / NCV;           // value groups of set 0 own the first d-tiles, of set 1 the rest
    const int cs = dt / kDtPerSet;
    const u32x4 pb = u32x4{pw[cs][0], pw[cs][1], pw[cs][2], pw[cs][3]};
    u32x4 a = unpack_v<VLO>(r.vc, dt);
    if constexpr (VHI != 0)
      st.acc[dt] = mma<BFV>(unpack_v<VHI>(r.vc + 2 * VLO, dt), u32x4{pwh[cs][0], pwh[cs][1], pwh[cs][2], pwh[cs][3]}, st.acc[dt]);
    if constexpr (RAWV && MASKED) {               // unquantized garbage may be Inf/NaN: clear the slots beyond seq_len
      uint32_t* aw = reinterpret_cast<uint32_t*>(&a);
#pragma unroll
      for (int v = 0; v < 4; ++v) aw[v] &= (valid[2 * v] ? 0x0000FFFFu : 0u) | (valid[2 * v + 1] ? 0xFFFF0000u : 0u);
    }
    st.acc[dt] = mma<BFV>(a, pb, st.acc[dt]);
    if constexpr (BFV) st.acc[dt] = mma<BFV>(a, u32x4{pl[0], pl[1], pl[2], pl[3]}, st.acc[dt]);
  }
}

// Record layout in the workspace: [b][hq][split] x (kHeadDim + 4) floats = acc[128], m, l, 0, 0.
constexpr int kRec = kHeadDim + 4;

// Fused decode step, first half: quantize the one new token of this (b,h) and store it at row t of the planes.  The
// first 16 lanes take the key row, the next 16 the value row (8 channels per lane; `raw` holds the lane's 16 input
// bytes, loaded by the caller).  Same arithmetic and bytes as the bulk quantize-append kernel.  The key codes and both
// scale/zero entries go to memory from here; the value codes go to `vstage` (128 bytes of LDS), from where the threads
// that own the block's words insert them after a barrier.  The reconstructed rows (code * scale + zero, one rounding as
// in App. B "Dequantization") go to `hat` (LDS: 128 key elements, then 128 value elements): the new token joins the
// attention from there, not from the cache.  bh: stream index in the planes (0 when paged: t is then a row number in
// plane order); sbh: the (batch, kv head) pair, for the stream's largest value-scale exponent.
template <int BK, int BV>
__device__ __forceinline__ void append_one(const DecodeArgs& a, int bh, int sbh, int tid, u32x4 raw, uint8_t* vstage, int64_t t,
                                           float* hat) {
  const Geom& g = a.g;
  const bool is_v = tid >= 16;
  const int lane16 = tid & 15, d0 = lane16 * 8;
  const uint32_t rw[4] = {raw.x, raw.y, raw.z, raw.w};
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), a.in_bf16);
  if (g.rotate_k | g.rotate_v) {                   // both 16-lane rows run the butterflies; a row that is not rotated
    float xr[8];                                   // keeps its own numbers
#pragma unroll
    for (int e = 0; e < 8; ++e) xr[e] = x[e];
    rotate8(xr, lane16, is_v ? rot_sign_bits(g.signs_v, lane16) : rot_sign_bits(g.signs_k, lane16));
    const bool take = is_v ? g.rotate_v != 0 : g.rotate_k != 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = take ? xr[e] : x[e];
  }
  uint32_t codes[8];
  uint16_t S, Z;
  const int bits = is_v ? BV : BK;
  const int G = is_v ? g.g_v : g.g_k, ng = is_v ? g.ng_v : g.ng_k;
  const int lpg = G >> 3;
  quantize8(x, bits, lpg, codes, &S, &Z);
  if (is_v && (lane16 & (lpg - 1)) == 0) note_value_scale(a.cache.v_scale_exp + sbh, S);
  // (picked by integer arithmetic: a per-lane choice among pointers of the argument block becomes a lookup in private memory)
  const uintptr_t km = reinterpret_cast<uintptr_t>(a.cache.k_meta) + (uintptr_t)((int64_t)bh * g.km_stream);
  const uintptr_t vm = reinterpret_cast<uintptr_t>(a.cache.v_meta) + (uintptr_t)((int64_t)bh * g.vm_stream);
  const uintptr_t meta = km + (is_v ? vm - km : (uintptr_t)0);
  if ((lane16 & (lpg - 1)) == 0)
    store_global<uint32_t>(meta + 4 * (uintptr_t)meta_index(t, lane16 >> lpg_shift(lpg), ng), (uint32_t)S | ((uint32_t)Z << 16));
  if (!is_v) {
    store_key_codes<BK>((uint8_t*)a.cache.k_codes + (int64_t)bh * g.kc_stream + t * (16 * BK), lane16, codes);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) vstage[d0 + e] = (uint8_t)codes[e];
  }
  const float sc = widen16(S, false), zp = widen16(Z, false);
#pragma unroll
  for (int e = 0; e < 8; ++e) hat[(is_v ? kHeadDim : 0) + d0 + e] = fmaf((float)code_value(codes[e]), sc, zp);   // (exact product: one rounding)
}

// The same for the slots of a residual buffer, which hold the rows as they came: 16 bytes per lane of the key row, and the
// value row's patterns at their places in the token's 32-token block.
__device__ __forceinline__ void append_patterns(const uint8_t* key_row, uintptr_t vblk, int u, int lane, u32x4 raw, bool bf16, float* hat) {
  const bool is_v = lane >= 16;
  const int d0 = 8 * (lane & 15);
  const uint32_t rw[4] = {raw.x, raw.y, raw.z, raw.w};
  if (!is_v) {
    store_global<u32x4>(reinterpret_cast<uintptr_t>(key_row) + 2 * d0, raw);
  } else {
    int dw, bit;
    v_field(u, d0, 16, &dw, &bit);
#pragma unroll
    for (int e = 0; e < 8; ++e)
      store_global<uint16_t>(vblk + 4 * (uintptr_t)(dw + 4 * e) + (bit >> 3), (uint16_t)(rw[e >> 1] >> (16 * (e & 1))));
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) hat[(is_v ? kHeadDim : 0) + d0 + e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), bf16);
}

// ---- the tokens still in the residual buffer of a cache with channel-wise keys ------------------------------------------
// One wavefront takes 32 of them (tile 0 .. RL/32 - 1) as one masked step over the buffer's patterns, behind its own part of the
// flushed tokens, into a (maximum, sum, accumulator) record in LDS that the final merge adds to the wavefronts' own.  What
// the step loads comes straight from memory in operand order, the query (as it is: the buffer holds unrotated rows) too.
// It is one memory latency and some 150 vector instructions, for the most part beside wavefronts that still walk the flushed
// tokens.  A launch of its own over the buffer (and one to merge) cost 5 to 6 us: K4V2, rotated keys, a fused step with 37 tokens
// in the buffer, 8 x 8 heads x 8192 tokens of 4 query heads 23.8 us so, 18.1 now (16.9 without a buffer); of 8 query heads
// 26.1 and 20.6; 32 x 8 heads x 8192 tokens 60.9 and 54.6; 8 heads x 2048 tokens 15.0 and 9.4.  (8 tokens per wavefront
// in vector arithmetic in front of the walk: 20.4 us and, for 8 query heads, 25.4.)
//   n    tokens in the buffer (slots 0 .. n - 1), more than 32 tile
//   q    this kv head's r_act query rows
template <int R, bool BF>
__device__ __forceinline__ void buffer_step(const uint8_t* k_resid, const uint8_t* v_resid, const uint16_t* q, int r_act, int n,
                                            int tile, const LaneCtx& L, float kappa, float (&rec)[R][kHeadDim], float (&rec_m)[R],
                                            float (&rec_l)[R]) {
  const int h = L.c % R;
  const bool head_lane = L.c < R;                  // (one column per head; the others carry nothing)
  u32x4 qb[1][4];
  StepRegs<16, 16> r;
  const uintptr_t qp = reinterpret_cast<uintptr_t>(q) + (head_lane && h < r_act ? h * (2 * kHeadDim) : 0) + 16 * L.j;
  const uintptr_t kp = reinterpret_cast<uintptr_t>(k_resid) + (32 * tile + L.c) * (2 * kHeadDim) + k_lane_offset<16>(L.j);
  const uintptr_t vp = reinterpret_cast<uintptr_t>(v_resid) + tile * (512 * 16) + 16 * L.lane;
#pragma unroll
  for (int m = 0; m < 4; ++m) qb[0][m] = load_global<u32x4>(qp + 64 * m);
#pragma unroll
  for (int x4 = 0; x4 < 2; ++x4)
#pragma unroll
    for (int m = 0; m < 4; ++m)
      *reinterpret_cast<u32x4*>(r.kc[x4] + 4 * m) = load_global<u32x4>(kp + 16 * x4 * (2 * kHeadDim) + k_piece_stride<16>() * m);
#pragma unroll
  for (int k = 0; k < 8; ++k) *reinterpret_cast<u32x4*>(r.vc + 4 * k) = load_global<u32x4>(vp + 1024 * k);
#pragma unroll
  for (int m = 0; m < 4; ++m) qb[0][m] = head_lane && h < r_act ? qb[0][m] : u32x4{0u, 0u, 0u, 0u};
  WaveState<1> st;
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) st.acc[dt] = float4v{0.f, 0.f, 0.f, 0.f};
  st.m = kNegBig; st.headroom = 0.f;
#pragma unroll
  for (int v = 0; v < 4; ++v) { st.l[v] = 0.f; st.noff[v] = 0.f; st.zacc[0][v] = 0.f; }
  const float qsum[1] = {0.f};
  NoKSeq none;
  compute_step<16, 16, R, BF, 1, 1, true>(r, qb, qb, qsum, kappa, st, L, tile, n, none);
  float l = (st.l[0] + st.l[1]) + (st.l[2] + st.l[3]);
  l = rows_sum(l);
  if (head_lane) {
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) *reinterpret_cast<float4v*>(&rec[h][16 * dt + 4 * L.j]) = st.acc[dt];
    if (L.j == 0) { rec_m[h] = st.m; rec_l[h] = l; }
  }
}

// Second half of the fused append: thread d < 128 inserts channel d's code of the new token into its 32-bit word of
// the 32-token block (the other fields of the word belong to other tokens of the block and keep their bits).  With
// 2-bit fields channels d and d+16 share a word (with 1-bit fields d, d+16, d+32 and d+48), so the thread of the first
// of those 16-channel tiles owns the word.  The word is loaded at the top of the kernel (field_word), long before the
// codes exist, and stored from here.  `shift`: the field is bits [shift, shift + B) of the staged code.
template <int B> constexpr int field_tiles() { return B == 1 ? 4 : B == 2 ? 2 : 1; }   // 16-channel tiles per word
template <int B> __device__ __forceinline__ bool field_owner(int tid) {
  return tid < kHeadDim && !((tid >> 4) & (field_tiles<B>() - 1));
}
template <int B> __device__ __forceinline__ int field_word(int tid, int u) {
  int dw, bit;
  v_field(u, tid & (kHeadDim - 1), B, &dw, &bit);
  return dw;
}
template <int B>
__device__ __forceinline__ uint32_t field_insert(uint32_t w, int tid, const uint8_t* vstage, int u, int shift) {
  const uint32_t fmask = (1u << B) - 1u;
#pragma unroll
  for (int f = 0; f < field_tiles<B>(); ++f) {
    int dwf, bitf;
    v_field(u, tid + 16 * f, B, &dwf, &bitf);             // same word, the neighbouring tiles' fields
    w = (w & ~(fmask << bitf)) | ((((uint32_t)vstage[tid + 16 * f] >> shift) & fmask) << bitf);
  }
  return w;
}

// One output element in the caller's type (16-bit types: rounded once).
__device__ __forceinline__ void store_out(void* out, int out_dtype, int64_t i, float val) {
  if (out_dtype == KVQ_F32) ((float*)out)[i] = val;
  else if (out_dtype == KVQ_F16) ((_Float16*)out)[i] = (_Float16)val;
  else ((uint16_t*)out)[i] = (uint16_t)bf16_rne(val);
}
// Partial records travel between workgroups that may sit on different parts of the chip, each with a cache of its own:
// their stores and loads are device-scope atomic accesses (performed where every compute unit sees them).
__device__ __forceinline__ void store_device(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_device(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Final output of rotated values: the normalized row sits in the rotated basis (LDS, 128 floats); 16 threads take it
// back with R_v^T (8 channels each) and store it in the output type.
__device__ __forceinline__ void store_unrotated_row(const float* row, int lane16, const uint32_t signs[4], void* out,
                                                    int out_dtype, int64_t hq) {
  float x[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) x[e] = row[8 * lane16 + e];
  unrotate8(x, lane16, rot_sign_bits(signs, lane16));
  const int64_t o = hq * kHeadDim + 8 * lane16;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (out_dtype == KVQ_F32) ((float*)out)[o + e] = x[e];
    else if (out_dtype == KVQ_F16) ((_Float16*)out)[o + e] = (_Float16)x[e];
    else ((uint16_t*)out)[o + e] = f32_to_bf16_bits(x[e]);
  }
}

// ---- sequences of different lengths: which part of which sequence a workgroup takes ------------------------------------
// A launch planned for the longest sequence cuts every sequence at the same places, and the workgroups behind a short one's
// end have nothing to do while those of the longest run on.  Instead all workgroups of a kv head (slots 0 .. slots - 1)
// are dealt out by the lengths: sequence b gets ceil(N_b / q) of them, q steps each, with the smallest q (a multiple of the wavefronts,
// and no more parts than kDealParts for the longest sequence, whose records one workgroup merges) for which they are enough.  Every wavefront works that out for itself from the lengths (at
// most 64, one per lane); the answer depends on nothing else, so all workgroups agree.  Where q would not come down to what pays
// (q_pay, from the plan: deal_pays), the plan's q stays, without the search.  One pass over the lanes counts the parts of both.
__device__ __forceinline__ int wave_scan(int v) {  // sum over the lanes up to and including this one
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);     // row_shr 1, 2, 4, 8
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);     // row_bcast 15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);     // row_bcast 31 into rows 2 and 3
  return v;
}
// (9 x 8 heads, one sequence of 12000 tokens among others of 1200, K4V2, in 16 parts 13.1 us, in 10 12.2; K8V8, 7 x 8, one of 16000, in 11 parts
// 22.1, in 17 19.1)
constexpr int kDealParts = 12;
struct Share { int b, split, count, q, slot0, len; };   // sequence, part of it, its parts, steps per part, slot of its first part, tokens
template <int UNIT, int MOST>                      // q is a multiple of UNIT steps (a workgroup's wavefronts); MOST: parts of the longest sequence
__device__ __forceinline__ Share balanced_share(const int32_t* __restrict__ seq_lens, int offset, int bound, int batch, int slots,
                                                int splits, int q_max, int q_pay, int slot, int lane) {
  const int len = min(max(seq_lens[min(lane, batch - 1)] + offset, 1), bound);
  const int n = lane < batch ? (len + 31) >> 5 : 0;           // steps, 2^19 at most
  // parts of q steps; (n + q - 1) / q in binary32: half a unit above the quotient of integers below 2^21 rounds to the right side
  auto parts = [&](int q) {
    const float rq = __builtin_amdgcn_rcpf((float)q);
    return (int)fmaf((float)(n + q - 1), rq, 0.5f * rq);
  };
  Share s;
  s.q = q_max;                                     // (always enough: no sequence is longer than the plan's)
  // (up to 4 parts of q_max a sequence, and q_pay is at least an eighth of it: 64 sequences count to 2048)
  const int both = wave_scan(parts(q_max) | parts(q_pay) << 16);
  int end = both & 0xFFFF, mine = parts(q_max);
  if (__builtin_amdgcn_readlane(both, 63) >> 16 <= slots) {   // (uniform)
    int lo = min(((splits * q_max + MOST - 1) / MOST + UNIT - 1) / UNIT, q_pay / UNIT), hi = q_pay / UNIT;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (__builtin_amdgcn_readlane(wave_scan(parts(mid * UNIT)), 63) <= slots) hi = mid; else lo = mid + 1;
    }
    s.q = hi * UNIT;
    mine = parts(s.q); end = wave_scan(mine);
  }
  const unsigned long long hit = __ballot(slot >= end - mine && slot < end);       // (one lane, or none)
  const int l = hit ? __ffsll(hit) - 1 : 0;
  s.b = hit ? l : -1;
  s.count = __builtin_amdgcn_readlane(mine, l);
  s.slot0 = __builtin_amdgcn_readlane(end, l) - s.count;
  s.split = slot - s.slot0;
  s.len = __builtin_amdgcn_readlane(len, l);
  return s;
}

// KSEQ: channel-wise keys (the caller passes the flushed part of the sequence: seq_len is a multiple of 64; the tokens in
// the residual buffer come on top, see buffer_step, and a fused step's token goes there); a wavefront then walks whole 64-token blocks (pairs of steps), rebuilding its query operands per block.
// PAGED: the planes are pools of pages; a step's data is found through this sequence's row of the page table.
// ROTV: the values are stored rotated (quantized caches with token-wise keys; compute_step then corrects its weights).
// HALF: at most 8 columns, two tiles side by side (sum_over_groups_half).
template <int BK, int BV, int R, int NW, bool BF, int NCK, int NCV, bool KSEQ = false, bool PAGED = false, bool ROTV = false, bool HALF = false>
__global__ __launch_bounds__(64 * NW, KVQ_WAVES_PER_SIMD) void decode_kernel(const DecodeArgs a) {
  constexpr int kSetGroups = 16 / R;             // groups per column set
  constexpr bool RAWK = BK == 16, RAWV = BV == 16;     // a tensor kept as its 16-bit patterns (either one, or both)
  constexpr bool RAW = RAWK;                          // (what the key side and the query staging ask)
  static_assert(!KSEQ || (!RAWK && !RAWV && NCK == 1), "channel-wise keys: quantized, one key column per head");
  static_assert(!ROTV || (!RAWK && !RAWV), "rotated values: both tensors quantized");
  constexpr int kRing = ring_stages<BK, BV, NCK, NCV, ROTV, HALF>();
#ifndef KVQ_KSEQ_STAGES
#define KVQ_KSEQ_STAGES 2
#endif
  // (channel-wise keys: the rebuild leaves registers for two steps, and the kernel, bound by its vector instructions,
  // measures no faster with a deeper ring)
  constexpr int kStages = KSEQ ? (kRing < KVQ_KSEQ_STAGES ? kRing : KVQ_KSEQ_STAGES) : kRing;
  constexpr int SPB = KSEQ ? 2 : 1;              // steps a wavefront takes in a row
  // codes enter the matrix unit as binary16 subnormals (code x 2^-24): the key side's factor goes into the logits'
  // scale, the value side's into the final accumulator
  constexpr float kUnit = RAWK ? 1.0f : kCodeUnit, kInvUnit = RAWK ? 1.0f : kInvCodeUnit;
  constexpr float kInvUnitV = RAWV ? 1.0f : kInvCodeUnit;
  // a wavefront's output rows at the end; until then the wavefront's own copy of the query (see "query" below)
  __shared__ __attribute__((aligned(16))) float sm_o[NW][R][kHeadDim];
  __shared__ float sm_m[NW][R], sm_l[NW][R];
  __shared__ __attribute__((aligned(16))) uint8_t sm_meta[NW][1024];
  __shared__ __attribute__((aligned(16))) float sm_zero[KSEQ ? kHeadDim : 16];   // query of a column that carries nothing
  __shared__ uint8_t sm_vnew[kHeadDim];          // fused step: the new token's value codes,
  __shared__ float sm_hat[2][kHeadDim];           // its reconstructed key and value rows,
  __shared__ float sm_mnew[R];                    // and its logit per head in log2 units
  __shared__ float sm_qsum[NW][R][4];
  __shared__ int sm_turn[NW];                      // how far each wavefront has come (see the main loop)
  // channel-wise keys: the records of the tokens still in the residual buffer (buffer_step: at most 128 of them)
  __shared__ __attribute__((aligned(16))) float sm_buf[KSEQ ? 4 : 1][R][kHeadDim];
  __shared__ float sm_bufm[KSEQ ? 4 : 1][R], sm_bufl[KSEQ ? 4 : 1][R];
  const Geom& g = a.g;
  const kvq_cache& cache = a.cache;
  const uint16_t* __restrict__ q = a.q;
  const int q_bf16 = a.q_bf16, q_heads = a.q_heads, out_dtype = a.out_dtype;
  const float softmax_scale = a.softmax_scale;
  float* __restrict__ ws = a.ws;
  void* __restrict__ out = a.out;

  // One word out of every cache line of the argument block, so that all of its lines are on their way at once: its fields are
  // first needed at four places down the chain that ends in the ring's first loads, and each waited for lines of its own (fused
  // steps, K4V2: 8 heads x 1024 tokens 8.17 us without and 7.83 with it, 8 x 8 heads x 8192 tokens 16.26 and 15.92,
  // 32 x 8 x 8 heads x 1024 tokens 11.30 and 11.03).
  {
    constexpr int kLines = (sizeof(DecodeArgs) + 63) / 64;
    static_assert(kLines <= 6 && sizeof(DecodeArgs) % 4 == 0, "argument block");
    const uint32_t* words = reinterpret_cast<const uint32_t*>(&a);
    uint32_t w[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) w[i] = words[min(16 * i, (int)(sizeof(DecodeArgs) / 4) - 1)];
    asm volatile("" :: "s"(w[0]), "s"(w[1]), "s"(w[2]), "s"(w[3]), "s"(w[4]), "s"(w[5]));
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int split = blockIdx.x, b = blockIdx.z;
  const int hk = blockIdx.y;
  int steps_per_split = a.steps_per_split;
  // this (batch, kv head)'s records: where the first lies and how far apart they are, this workgroup's one, and whether it
  // is the only one (its result then goes straight to the output)
  int n_rec = a.rec_splits, slot = 0, slot0 = 0;
  int seq_len = a.seq_len;
  int n_buf = a.buf_len;                           // channel-wise keys: this sequence's tokens in the residual buffer
  bool have_len = a.seq_lens == nullptr;
  if constexpr (!KSEQ) {
    if (a.balance) {                               // (uniform)
      slot = b;
      const Share sh = balanced_share<NW, BK + BV <= 8 ? kDealParts : 2 * kDealParts>(a.seq_lens, a.lens_offset, a.lens_bound, g.batch, a.balance, a.n_splits, a.steps_per_split, a.deal_pays, slot, lane);
      if (sh.b < 0) return;                        // more workgroups than parts
      b = sh.b; split = sh.split; steps_per_split = sh.q; n_rec = sh.count; slot0 = sh.slot0;
      seq_len = sh.len; have_len = true;
    }
  }
  const int bh = b * g.kv_heads + hk;
  // this sequence's length: its own when the caller gave per-sequence lengths, inside what the launch was planned for
  if (!have_len) {
    int n = min(max(a.seq_lens[b] + a.lens_offset, 1), a.lens_bound);
    n_buf = n & (a.lens_block - 1);
    if (a.lens_mode == 1) n &= ~(a.lens_block - 1);         // a residual buffer of lens_block slots: the flushed blocks ...
    else if (a.lens_mode == 2) n &= a.lens_block - 1;       // ... or the tail in the buffer (either may be empty)
    seq_len = min(n, a.seq_len);
  }

  std::conditional_t<ROTV, LaneCtxRotV, LaneCtx> L;
  L.lane = lane; L.c = lane & 15; L.j = lane >> 4;
  L.ngk = g.ng_k; L.ngv = g.ng_v;
  constexpr int kHalfGroups = 8 / R;
  const int h = HALF ? (L.c & 7) / kHalfGroups : L.c % R, grp = HALF ? (L.c & 7) % kHalfGroups : L.c / R;
  const bool act_k = grp < g.ng_k, act_v = grp < g.ng_v;
  L.gk = act_k ? grp : 0; L.gv = act_v ? grp : 0;
  const int64_t bh_base = PAGED ? 0 : bh;           // paged: rows are numbered from the plane base (virtual_token)
  L.kc = (const uint8_t*)cache.k_codes + bh_base * g.kc_stream;
  L.vc = (const uint8_t*)cache.v_codes + bh_base * g.vc_stream;
  L.kc_off = L.c * (16 * BK) + k_lane_offset<BK>(L.j);
  L.vc_off = lane * (BV == 1 ? 8 : 16);
  {
    // channel-wise keys: 512 bytes of scale/zero per group of seq_g = 32, 64 or 128 tokens (32 lanes), fetched with
    // every step of the group (1, 2 or 4 of them)
    const int nk = RAWK ? 0 : KSEQ ? 32 : 8 * g.ng_k, nv = RAWV ? 0 : 8 * g.ng_v;   // (an unquantized tensor has none)
    const int ml = min(lane, nk + nv - 1);       // lanes beyond the scale/zero bytes of a step repeat the last 16
    const bool is_k = ml < nk;
    L.meta_base = is_k ? (const uint8_t*)cache.k_meta + bh_base * g.km_stream
                       : (const uint8_t*)cache.v_meta + bh_base * g.vm_stream;
    L.meta_mul = is_k ? (KSEQ ? 16384 >> __builtin_ctz(g.seq_g | 16384) : 128 * g.ng_k) : 128 * g.ng_v;
    L.meta_off = 16 * (is_k ? ml : ml - nk);
    L.meta_step_mask = (KSEQ && is_k) ? ~(uint32_t)((g.seq_g >> 5) - 1) : ~0u;
    L.km_rd = (L.gk * 16 + 4 * L.j) * 4;                       // key bytes come first in the LDS copy
    L.vm_rd = 16 * nk + (L.gv * 16 + 4 * L.j) * 4;
    if constexpr (HALF) {                                      // (this half's tile)
      L.km_rd += (L.c >> 3) * 64 * L.ngk;
      L.vm_rd += (L.c >> 3) * 64 * L.ngv;
    }
    L.meta_lds = &sm_meta[wave][0];
  }

  // ---- what this launch reads.  A fused decode step does not read its new token (position seq_len - 1) back from the
  // cache: the workgroup that owns that position quantizes and stores it, and adds it to the attention as one more
  // partial record, computed from the reconstruction it holds in registers (no store -> load round trip, no fence).
  // (Both tensors unquantized: the kernel that reads residual buffers.  The new token then goes to its slot as it is.)
  // (Channel-wise keys: the sequence's last workgroup takes the tokens in the residual buffer as well, n_buf of them, and the
  // new token goes there as it is.)
  constexpr bool kCanAppend = RAWK == RAWV;
  const bool fused = kCanAppend && a.k_new != nullptr;
  const int n_att = fused && !KSEQ ? seq_len - 1 : seq_len;        // tokens attended through the cache planes
  const int n_steps = (n_att + 31) >> 5;
  const int step_begin = split * steps_per_split;
  const int step_end = min(step_begin + steps_per_split, n_steps);
  const bool last_split = KSEQ ? split == a.n_splits - 1 : (unsigned)(((seq_len + 31) >> 5) - 1 - step_begin) < (unsigned)steps_per_split;
  const bool do_append = fused && last_split;             // uniform over the workgroup
  // this wavefront's steps: step_begin + wave, + NW, ...; the last one may be the ragged tail of the sequence
  const int first = step_begin + SPB * wave;
  auto step_of = [&](int i) { return KSEQ ? first + 2 * NW * (i >> 1) + (i & 1) : first + NW * i; };
  const int n_my = first < step_end ? SPB * ((step_end - first + SPB * NW - 1) / (SPB * NW)) : 0;
  const bool ragged = (n_att & 31) != 0;
  const bool own_tail = ragged && n_my > 0 && step_of(n_my - 1) == n_steps - 1;
  const int n_full = own_tail ? n_my - 1 : n_my;   // complete steps of this wavefront
  // A step that is always there to load from: wavefronts with nothing to do still issue the ring's loads (see refill).
  const int safe_step = min(step_begin, max(n_steps - 1, 0));
  // paged: logical step -> step number in plane order (page of the pool, this head's share of it, step inside it).  The
  // page numbers of a wavefront's own steps are copied to LDS by the wavefront first: one is needed before every step's
  // loads can be issued, and a global load in front of them costs the ring most of its depth.
  constexpr int kPageSlots = PAGED ? 512 : 1;    // (steps of one wavefront; a longer walk reads the table itself)
  __shared__ int32_t sm_pages[PAGED ? NW : 1][kPageSlots];
  const int32_t* __restrict__ my_pages = PAGED ? cache.page_table + (int64_t)b * g.pages_per_seq : nullptr;
  const int step_shift = g.page_shift - 5;
  if constexpr (PAGED) {
    for (int i = lane; i < min(n_my, kPageSlots); i += 64) sm_pages[wave][i] = my_pages[step_of(i) >> step_shift];
    if (n_my == 0 && lane == 0) sm_pages[wave][0] = my_pages[safe_step >> step_shift];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
  // (i: the step's place in the wavefront's walk)
  // The two places a page number may come from are two loads with a wait of their own, the table's named as global memory: written as
  // one choice of places they became one flat load, and its use waits for everything in flight, i.e. the ring was drained in every step.
  // In turn, that way and this: 16 sequences of 600 to 16001 tokens, 8 kv heads, K4V2 30.0 and 28.9 us, K4V4 31.5 and 31.4; 32 sequences of
  // 16000 to 16384 tokens, 64 query heads, K4V2 79.3 and 77.8; 4 of 24866 to 74598, 24 query heads, K3V2 48.2 and 46.1.
  auto fetch = [&](StepRegs<BK, BV>& dst, int i, int step, uint32_t lane_mask) {
    if constexpr (PAGED) {
      int32_t page;                              // (uniform)
      if (i < kPageSlots) page = __builtin_amdgcn_readfirstlane(sm_pages[wave][i]);
      else page = __builtin_amdgcn_readfirstlane(load_global<int32_t>(reinterpret_cast<uintptr_t>(my_pages + (step >> step_shift))));
      load_step<BK, BV, true>(dst, L, (((int64_t)page * g.kv_heads + hk) << step_shift) + (step & ((1 << step_shift) - 1)), lane_mask);
    } else {
      load_step<BK, BV>(dst, L, step, lane_mask);
    }
  };

  // ---- the small loads of the prologue go first, so that they return ahead of the ring's first fill: the query rows (every
  // wavefront loads them all; lanes beyond the rows re-read the first 16 bytes), and in the wavefront that appends a fused
  // step's token that token's rows and the words of the value block that take its codes (lanes that have none of these re-read the query).
  // Those are issued in front of every load of the ring and used by that wavefront alone, so a branch around them costs no
  // load its count, and the others save their addresses (K4V2, 4 to 8 heads x 1024 to 2048 tokens 0.05 to 0.1 us of 7.3 to 8.5).
  int stream_scale_exp = 0;                        // largest exponent field of the stream's value scales (weight_headroom)
  if constexpr (!RAWV) stream_scale_exp = cache.v_scale_exp[bh];
  const int r_act = a.heads_per_kv;                // heads that exist (R is the next power of two)
  constexpr int kQItems = R > 4 ? 2 : 1;           // 16-byte pieces of the query rows per lane: item lane + 64 t
  const uint16_t* qbase = q + ((int64_t)b * q_heads + hk * r_act) * kHeadDim;
  u32x4 qraw[kQItems];
#pragma unroll
  for (int t = 0; t < kQItems; ++t) {
    const int item = lane + 64 * t;
    qraw[t] = *reinterpret_cast<const u32x4*>(qbase + (item < R * 16 && (item >> 4) < r_act ? item * 8 : 0));
  }
  // The fused append is one wavefront's work: of 8 the fourth's.  Wavefronts 0-3 are a microsecond ahead of 4-7, which share their SIMDs,
  // when the first step's data comes; the last one, which had it before (it has a step less where the steps do not divide
  // evenly), brought that and the append to the final barrier.  Fused steps with the last and with the fourth wavefront's append, in turn, K4V2:
  // 8 heads x 1024 tokens, 1 query head, 8.88 and 8.48 us, 4 query heads 9.02 and 8.50; 8 x 8 heads x 2048 tokens 10.27
  // and 9.47 (9.27 without an append), x 8192 16.75 and 16.64; 32 x 8 x 8 heads x 1024 tokens 12.44 and 11.91.
  constexpr int VLO_ = v_lo<BV>(), VHI_ = v_hi<BV>();
  const bool app_wave = do_append && wave == (NW == 8 ? 3 : NW - 1);
  u32x4 nraw = u32x4{0u, 0u, 0u, 0u};
  uint32_t vw_lo[2] = {0u, 0u}, vw_hi[2] = {0u, 0u};
  uintptr_t vblk = 0;                              // the new token's 32-token block of value codes
  int64_t t_new = 0;
  int u_new = 0;                                   // its place in that block
  if constexpr (kCanAppend) {
    if (app_wave) {                                // uniform
      // (paged: the new token's row number in plane order, with the stream index 0)
      if constexpr (KSEQ) {
        t_new = n_buf - 1;                         // its slot in the buffer
      } else if constexpr (PAGED) {
        const int64_t pg = my_pages[(seq_len - 1) >> g.page_shift];
        t_new = ((pg * g.kv_heads + hk) << g.page_shift) + ((seq_len - 1) & ((1 << g.page_shift) - 1));
      } else {
        t_new = seq_len - 1;
      }
      // (the address is picked by integer arithmetic: a per-lane choice among pointers held in the argument block would
      // be turned into a lookup in private memory)
      const int64_t row_off = ((int64_t)b * a.nsb + (int64_t)hk * a.nsh + (lane & 15) * 8) * 2;
      const uintptr_t qp = reinterpret_cast<uintptr_t>(qbase), kp = reinterpret_cast<uintptr_t>(a.k_new),
                      vp = reinterpret_cast<uintptr_t>(a.v_new);
      const uintptr_t nsrc = qp + (lane < 32 ? (kp - qp) + (lane >= 16 ? vp - kp : (uintptr_t)0) + (uintptr_t)row_off : (uintptr_t)0);
      nraw = load_global<u32x4>(nsrc);
      if constexpr (KSEQ)
        vblk = reinterpret_cast<uintptr_t>(cache.v_resid) + (uintptr_t)((int64_t)bh * g.resid * (2 * kHeadDim) + (t_new >> 5) * (int64_t)(512 * 16));
      else
        vblk = reinterpret_cast<uintptr_t>(cache.v_codes) + (uintptr_t)(bh_base * g.vc_stream + (t_new >> 5) * (int64_t)(512 * BV));
      u_new = (int)(t_new & 31);
      if constexpr (!RAWV && !KSEQ) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {              // channels lane and lane + 64
          const bool own_lo = field_owner<VLO_>(lane + 64 * t);
          vw_lo[t] = load_global<uint32_t>(qp + (own_lo ? vblk - qp + 4 * (uintptr_t)field_word<VLO_>(lane + 64 * t, u_new) : (uintptr_t)0));
          if constexpr (VHI_ != 0) {
            const bool own_hi = field_owner<VHI_>(lane + 64 * t);
            vw_hi[t] = load_global<uint32_t>(qp + (own_hi ? vblk - qp + 4 * (uintptr_t)(128 * VLO_ + field_word<VHI_>(lane + 64 * t, u_new)) : (uintptr_t)0));
          }
        }
      }
    }
  }

  // ---- register ring of kStages steps, filled right away.
  // Ring slot k is refilled with the wavefront's i-th step (the ragged tail included); past its last step the loads
  // are still issued, at that last step (or at safe_step for a wavefront that has none) and collapsed to one cache line
  // each (see load_step), so that no load of the ring is conditional.
  StepRegs<BK, BV> buf[kStages];
  auto refill = [&](int k, int i) {
    const int ic = max(min(i, n_my - 1), 0);
    fetch(buf[k], ic, n_my > 0 ? step_of(ic) : safe_step, i < n_my ? ~0u : 0u);
  };
  // Only the first half of the ring goes out in front of the query staging: the memory pipeline of a compute unit
  // takes in about what two steps of eight wavefronts ask for, and a wavefront that issues more waits at the load until
  // earlier data has come back.  The second half follows the staging, by when the first is on its way out of memory.
  constexpr int kEarly = (kStages + 1) / 2;
#pragma unroll
  for (int k = 0; k < kEarly; ++k) refill(k, k);

  // ---- query: every wavefront stages the rows for itself, in its own part of sm_o, already in the form its lanes want
  // them in -- the matrix operands of the key side (binary16, divided by the slots' position factors, in operand order;
  // the unquantized kernel: the patterns themselves), or for channel-wise keys binary32 rows -- so that no barrier
  // stands between a wavefront's first loads and its first step, and a lane converts its own 8 channels and no more.
  // What bounds a short launch is this chain of latencies.  Fused steps with the rows staged once per workgroup (a
  // barrier that waited for the first half of the ring, then every lane built its operands from 32 channels; the append
  // spread over two wavefronts) and like this: 1024 tokens of 8 heads 10.4 and 9.2 us, the 8B layer at B=8 and 8192
  // tokens 19.9 and 18.3, 8 x 64 heads x 2048 tokens 14.5 and 12.6; the 70B layer, where the chain is 2 % of the step, 150.8
  // and 150.6.
  constexpr int KLO = k_lo<BK>(), KHI = k_hi<BK>();
  constexpr int kOpRow = KHI != 0 ? 512 : 256;     // bytes of one head's staged operands: [j][m][slot], the high run's behind
  uint8_t* const q_lds = reinterpret_cast<uint8_t*>(&sm_o[wave][0][0]);
  bool q_is_bf16 = q_bf16 != 0;
  float xq[kQItems][8];                            // this lane's channels of the staged rows
  {
    typedef u32x4 __attribute__((may_alias)) u32x4_lds;
    typedef uint16_t __attribute__((may_alias)) u16_lds;
    typedef float4v __attribute__((may_alias)) f32x4_lds;
    constexpr int kZeroBytes = KSEQ ? 512 : 64;
    if (lane < kZeroBytes / 16) reinterpret_cast<u32x4_lds*>(sm_zero)[lane] = u32x4{0u, 0u, 0u, 0u};   // (every wavefront: the same)
#pragma unroll
    for (int t = 0; t < kQItems; ++t) {
      const int item = lane + 64 * t, hh = item >> 4, o = item & 15;
      const bool have = hh < r_act;                // a surplus head is an all-zero query: uniform weights, never stored
      const u32x4 raw = have ? qraw[t] : u32x4{0u, 0u, 0u, 0u};
      const uint32_t rw[4] = {raw.x, raw.y, raw.z, raw.w};
      if constexpr (RAWK) {
        if (item < R * 16) *reinterpret_cast<u32x4_lds*>(q_lds + hh * 256 + (o & 3) * 64 + (o >> 2) * 16) = raw;
#pragma unroll
        for (int e = 0; e < 8; ++e) xq[t][e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), q_is_bf16);   // (a fused step's logit)
      } else {
        float xk[8];
        float (&x)[8] = *(KSEQ ? &xk : &xq[t]);    // (the residual buffer holds rows as they came: their scores take the query as it is)
#pragma unroll
        for (int e = 0; e < 8; ++e) xq[t][e] = x[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), q_is_bf16);
        if (g.rotate_k) {
          // rotated keys: the scores need R q, rounded once to binary16 (16 lanes hold one query row, 8 channels each)
          rotate8(x, o, rot_sign_bits(g.signs_k, o));
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = widen16(f32_to_f16_bits(x[e]), false);
        }
        if constexpr (KSEQ) {
          if (item < R * 16) {
            f32x4_lds* dst = reinterpret_cast<f32x4_lds*>(q_lds + hh * 512 + o * 32);
            float y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = x[e] / (kseq_prescaled<BK>() ? k_chan_scale<BK>(e) : 1.0f);
            dst[0] = float4v{y[0], y[1], y[2], y[3]};
            dst[1] = float4v{y[4], y[5], y[6], y[7]};
          }
        } else {
          auto stage = [&](auto run, uint8_t* row) {           // the operand of one run of the codes: see k_octet_offset
            constexpr int B = decltype(run)::bits, BASE = decltype(run)::base;
            uint16_t y[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] = __builtin_bit_cast(uint16_t, (_Float16)(x[e] * (decltype(run)::factor / k_octet_scale<B, BASE>(e))));
            if constexpr (B == 4) {
              *reinterpret_cast<u32x4_lds*>(row + o * 16) = u32x4{y[0] | (uint32_t)y[4] << 16, y[1] | (uint32_t)y[5] << 16,
                                                                  y[2] | (uint32_t)y[6] << 16, y[3] | (uint32_t)y[7] << 16};
            } else if constexpr (B == 8) {
              *reinterpret_cast<u32x4_lds*>(row + o * 16) = u32x4{y[0] | (uint32_t)y[2] << 16, y[1] | (uint32_t)y[3] << 16,
                                                                  y[4] | (uint32_t)y[6] << 16, y[5] | (uint32_t)y[7] << 16};
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e) *reinterpret_cast<u16_lds*>(row + k_octet_offset<B>(o) + 16 * (e >> 2) + 4 * (e & 3)) = y[e];
            }
          };
          if (item < R * 16) {
            stage(KRun<KLO, k_default_base<KLO>(), 1>{}, q_lds + hh * kOpRow);
            if constexpr (KHI != 0) stage(KRun<KHI, k_hi_base<BK>(), (1 << KLO)>{}, q_lds + hh * kOpRow + 256);
          }
          // per-group sums of the (staged) query: the zero points of a key group enter the scores through them
          float part = 0.f;
#pragma unroll
          for (int e = 0; e < 8; ++e) part += x[e];
          const int lpg = g.g_k >> 3;              // lanes per key group: 4, 8 or 16
          part = lanes_sum(part, lpg);
          if (item < R * 16 && (o & (lpg - 1)) == 0) sm_qsum[wave][hh][o >> lpg_shift(lpg)] = part;
        }
      }
    }
  }
  // ---- fused step: one wavefront quantizes the new token (two 16-lane rows), stores keys and scale/zero, inserts the value
  // codes into their words (loaded at the top), and the new token becomes a partial record of its own: logit of every
  // head against the reconstructed key row (maximum = that logit, sum = one weight of 1, accumulator = the reconstructed
  // value row), which the merge below adds to the wavefronts' records.  All of it stays inside the wavefront.
  if constexpr (kCanAppend) {
    if (app_wave) {                                // uniform
      if constexpr (KSEQ) {
        const uint8_t* row = reinterpret_cast<const uint8_t*>(cache.k_resid) + ((int64_t)bh * g.resid + t_new) * (2 * kHeadDim);
        if (lane < 32) append_patterns(row, vblk, u_new, lane, nraw, a.in_bf16 != 0, &sm_hat[0][0]);
      } else if constexpr (RAWV) {
        if (lane < 32) append_patterns(L.kc + t_new * (2 * kHeadDim), vblk, u_new, lane, nraw, a.in_bf16 != 0, &sm_hat[0][0]);
      } else {
        if (lane < 32) append_one<BK, BV>(a, PAGED ? 0 : bh, bh, lane, nraw, sm_vnew, t_new, &sm_hat[0][0]);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if constexpr (!RAWV && !KSEQ)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int d = lane + 64 * t;
        if (field_owner<VLO_>(d))
          store_global<uint32_t>(vblk + 4 * (uintptr_t)field_word<VLO_>(d, u_new), field_insert<VLO_>(vw_lo[t], d, sm_vnew, u_new, 0));
        if constexpr (VHI_ != 0) {
          if (field_owner<VHI_>(d))
            store_global<uint32_t>(vblk + 4 * (uintptr_t)(128 * VLO_ + field_word<VHI_>(d, u_new)), field_insert<VHI_>(vw_hi[t], d, sm_vnew, u_new, VLO_));
        }
      }
#pragma unroll
      for (int t = 0; t < kQItems; ++t) {          // 16 lanes per head: 8 channels each, then a sum over the 16
        const int item = lane + 64 * t, o = item & 15;
        float part = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) part = fmaf(xq[t][e], sm_hat[0][8 * o + e], part);
        part = lanes_sum(part, 16);
        if (o == 0 && item < R * 16) sm_mnew[item >> 4] = part * (softmax_scale * kLog2e);
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int k = kEarly; k < kStages; ++k) refill(k, k);       // the second half of the ring's first fill
  // column c of set cs carries head h restricted to key group grp + cs*kSetGroups (zero elsewhere)
  u32x4 qb[NCK][4];
  u32x4 qbh[NCK][4];                             // operand of the high run of 3- and 6-bit key codes (else unused)
  float qsum_u[NCK];
#pragma unroll
  for (int cs = 0; cs < NCK; ++cs) {
    typedef u32x4 __attribute__((may_alias)) u32x4_lds;
    const int gcs = grp + cs * kSetGroups;
    const bool act = gcs < g.ng_k;
    const bool mine = act && (RAW || (32 * L.j) >> __builtin_ctz(g.g_k) == gcs);          // (unquantized: one group)
    const uint8_t* zero = reinterpret_cast<const uint8_t*>(sm_zero);
    const uint8_t* src = mine ? q_lds + h * kOpRow + L.j * 64 : zero;
    const uint8_t* src_hi = mine && KHI != 0 ? q_lds + h * kOpRow + 256 + L.j * 64 : zero;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      if constexpr (!KSEQ) {
        qb[cs][m] = *reinterpret_cast<const u32x4_lds*>(src + 16 * m);
        if constexpr (KHI != 0) qbh[cs][m] = *reinterpret_cast<const u32x4_lds*>(src_hi + 16 * m);
      }
    }
    float qsum = 0.f;
    if constexpr (!RAW && !KSEQ) { if (act) qsum = sm_qsum[wave][h][gcs]; }
    qsum_u[cs] = qsum * kUnit;
  }
  const float kappa = softmax_scale * kLog2e * kInvUnit;

  WaveState<NCV, HALF> st;
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) st.acc[dt] = float4v{0.f, 0.f, 0.f, 0.f};
  st.m = kNegBig;
  st.headroom = 0.f;
  if constexpr (!RAWV) st.headroom = weight_headroom<BV>(stream_scale_exp);
#pragma unroll
  for (int v = 0; v < st.kClasses; ++v) {
    st.l[v] = 0.f; st.noff[v] = 0.f;
#pragma unroll
    for (int cs = 0; cs < NCV; ++cs) st.zacc[cs][v] = 0.f;
  }

  // ---- main loop, unrolled over the ring: compute a step, then refill its registers with the step kStages
  // ahead, so that kStages-1 steps of loads are always in flight behind the one being computed.
  typename std::conditional<KSEQ, typename std::conditional<k_hi<BK>() != 0, KSeqState2, KSeqState>::type, NoKSeq>::type ks;
  const float* qrow = KSEQ && grp < 2 ? &sm_o[wave][h][0] : sm_zero;      // (column groups 0 and 1 carry the key side)
  // one complete step out of ring slot k (for channel-wise keys an even slot starts a 64-token block, and the query
  // operands are rebuilt there: once per group of 64 tokens, twice per group of 128 -- the second time from the same
  // entries -- and in the odd steps too when a group is one step long)
  const bool rebuild_every_step = KSEQ && g.seq_g == 32;       // (uniform)
  auto full_step = [&](int k, int i) {
    if constexpr (KSEQ) {                        // an even step of this wavefront's sequence starts a block (uniform;
      const int odd = kStages % 2 == 0 ? (k & 1) : (i & 1);      // with an even ring it is the ring slot's parity)
      compute_step<BK, BV, R, BF, NCK, NCV, false, true, HALF>(buf[k], qb, qbh, qsum_u, kappa, st, L, step_of(i), n_att, ks, qrow,
                                                         grp == 1 ? 1.0f : 0.0f, !odd || rebuild_every_step);
    } else {
      compute_step<BK, BV, R, BF, NCK, NCV, false, false, HALF>(buf[k], qb, qbh, qsum_u, kappa, st, L, step_of(i), n_att, ks);
    }
  };
  // the ragged tail of the sequence out of ring slot k (it came through the ring like every other step): masked
  auto tail_step = [&](int k) {
    if constexpr (!KSEQ)
      compute_step<BK, BV, R, BF, NCK, NCV, true, false, HALF>(buf[k], qb, qbh, qsum_u, kappa, st, L, n_steps - 1, n_att, ks);
  };
  // Two wavefronts share a SIMD (w and w + 4 of a workgroup of 8; of 4, two workgroups), and at equal priority it serves the
  // older one first: wavefronts 0-3 of the 70B layer's step were done after 103 us and 4-7 after 136, those of 8 x 8 heads x 8192
  // tokens after 9.0 and 12.3, and what a wavefront walks alone comes at half the rate.  So whoever is behind goes first.  Short
  // walks give their turns (kStages steps) falling priorities; from 4 turns on (8 steps, 12 of a ring of three) a wavefront notes each turn in LDS and goes
  // last where its partner has not come as far (a stale or early look costs a turn at the wrong priority, nothing else); a
  // workgroup of 4 does not know its partner and takes a priority per quarter of its walk.  In turn, K4V2, turns of four steps, before and with it:
  // 70B step 148.3 and 143.3 us, 8 x 8 heads x 32768 tokens 47.7 and 44.4, x 16384 26.1 and 25.3, x 8192 17.1 and 16.7, 32 x 8 x 8 heads x
  // 4096 tokens 25.9 and 24.9, 40 x 8 x 8 heads x 2000 tokens 22.2 and 21.3.  (Falling quarters for all 145.6, 45.6, 25.4, 16.8, 24.9; by the partner
  // for all 143.6, 44.3, 25.3, 17.3, 25.1; steps drawn from a counter in LDS 146.1, 44.2, 25.9, 17.4, 25.8: a wavefront draws
  // a ring ahead of what it computes, so the last steps still meet at the slow ones.)  By the partner from 8 steps on and only from 16, turns of two
  // steps, 56 fused steps of K4V2 and K4V4, 4 and 8 query heads, 1 to 32 sequences: 0.2 % slower in the mean from 16, 32 x 8 heads x 3600 tokens
  // 21.0 and 21.4 us (8 query heads 22.0 and 22.3), 16 x 8 x 4096 14.7 and 14.5.
  // Not where memory alone binds: the sum of the widths, and 8-bit keys with values of one run (K8V8, 8 x 8 heads x 32768 tokens: 85.5 us
  // before, 86.6 with it).  Equal priorities and these, 32 x 8 x 8 heads, in turn, means over eight placements of the planes (a call's time
  // differs by up to 8 % between them, above all where sequences lie powers of two apart): K8V2 x 24576 tokens 185.9 and 192.5,
  // x 36000 256.8 and 253.7, x 40960 299.7 and 321.8; K8V1 x 40960 287.0 and 305.4, K8V4 335.2 and 353.7, x 65536 522.4 and 519.9; 8 x
  // 8 heads x 8192 tokens K8V4 22.4 and 22.4, K8V3 22.1 and 21.8.  On this side of the line keys of up to 4 bits gain 1 to 6 % (K4V2 x 65536
  // 304.6 and 292.4, K4V4 377.6 and 362.5, K4V8 539.2 and 532.0, K1V8 395.6 and 384.8, K3V6 463.7 and 443.5).
  // 6-bit keys gain 1 to 4 % (K6V1 x 36000 205.6 and 197.5, K6V6 308.7 and 304.9; K6V3 anywhere, x 65536 469.6 and 452.4), except in long walks
  // over sequences that lie a power of two from 32768 tokens on apart, as they do in a cache of that capacity, whatever they are filled to:
  // there all turns have one priority.  Capacity 32768, 22937 tokens, K6V1 132.3 and 134.5, K6V6 192.2 and 196.4; capacity 65536, 13107 tokens (51
  // steps) K6V2 84.6 and 85.7, 29491 K6V2 177.8 and 186.3, K6V4 210.1 and 216.2; 16 x 8 sequences of 131072, 91750 tokens K6V1 263.7 and 281.7.
  // Not with a capacity of 16384 (K6V1 95.8 and 94.5) nor in shorter walks (8 x 8 sequences of 32768, 32 steps, K6V2 54.7 and 53.7).
  // Nor over channel-wise keys by 8 wavefronts (K4V2, 8 x 8 heads x 8229 tokens 17.25 and 17.44 us, K4V4 19.5 and 20.1; by 4, 40 x 8
  // heads x 3000 tokens, 33.3 and 32.3).
  constexpr bool kPairs = NW == 8, kYield = BK + BV <= 12 && !(BK == 8 && v_hi<BV>() == 0) && !(KSEQ && kPairs);
  const bool level = BK == 6 && BV != 3 && kPairs && !PAGED && n_full >= 48 && g.t_cap >= 32768 && (g.t_cap & (g.t_cap - 1)) == 0;
  const bool by_partner = kYield && kPairs && n_full >= 4 * kStages && !level;
  const int q1 = level ? n_full : kPairs ? kStages : n_full >> 2, q2 = level ? n_full : kPairs ? 2 * kStages : n_full >> 1, q3 = q1 + q2;
  int partner = 0;                                 // the turn that the other wavefront of this SIMD has reached, in steps
  if constexpr (kYield && kPairs) __hip_atomic_store(&sm_turn[wave], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if constexpr (kYield) __builtin_amdgcn_s_setprio(3);
  int it = 0;
  for (; it + kStages <= n_full; it += kStages) {
    if constexpr (kYield) {                        // (uniform, all of this)
      if (by_partner) {
        if (partner < it) __builtin_amdgcn_s_setprio(0); else __builtin_amdgcn_s_setprio(3);
      } else {
        if (it >= q3) __builtin_amdgcn_s_setprio(0);
        else if (it >= q2) __builtin_amdgcn_s_setprio(1);
        else if (it >= q1) __builtin_amdgcn_s_setprio(2);
      }
    }
#pragma unroll
    for (int k = 0; k < kStages; ++k) {
      if (kYield && kPairs && k == kStages - 1) {
        __hip_atomic_store(&sm_turn[wave], it + kStages, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        partner = __builtin_amdgcn_readfirstlane(__hip_atomic_load(&sm_turn[wave ^ (NW / 2)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
      }
      full_step(k, it + k);
      refill(k, it + k + kStages);
    }
  }
#pragma unroll
  for (int k = 0; k < kStages - 1; ++k) {        // the last few complete steps are already in the ring,
    if (it + k >= n_full) break;
    full_step(k, it + k);
  }
  if (own_tail) {                                 // and so is the tail, in the slot after them
    const int kt = n_full - it;
#pragma unroll
    for (int k = 0; k < kStages; ++k)
      if (kt == k) tail_step(k);
  }

  if constexpr (kYield) __builtin_amdgcn_s_setprio(0);
  // ---- channel-wise keys, the sequence's last workgroup: the tokens in the residual buffer, behind the totals below
  const int n_old = KSEQ && last_split ? n_buf - (fused ? 1 : 0) : 0;
  // ---- wavefront totals: l and zacc over register classes and the 4 lane groups j; then this lane's output rows
  float l = 0.f;
  const bool upper = HALF && (L.c & 8);
  // (of the lane's class: the halves' classes are two apart; then over both halves)
  auto class_factor = [&](int v) { return upper ? (float)(1 << v_slot_shift<BV>((v + 2) & 3)) : (float)(1 << v_slot_shift<BV>(v)); };
  auto both_halves = [&](float x) { return HALF ? x + __uint_as_float(halves_swap(__float_as_uint(x))) : x; };
#pragma unroll
  for (int v = 0; v < st.kClasses; ++v) l = fmaf(st.l[v], class_factor(v), l);
  l = both_halves(rows_sum(l));
#pragma unroll
  for (int cs = 0; cs < NCV; ++cs) {
    float z = 0.f;
#pragma unroll
    for (int v = 0; v < st.kClasses; ++v) z = fmaf(st.zacc[cs][v], class_factor(v), z);
    z = both_halves(rows_sum(z));
    const int gcs = grp + cs * kSetGroups;                     // the value group this lane's column carries in set cs
    if (gcs < g.ng_v && !upper) {
      // (a shift: group counts are powers of two, and eight divisions by them, with a group's tokens and the last step's owner in
      // the prologue, took 0.2 to 0.6 us of a launch: 8 heads x 1024 tokens 7.83 us with them, 7.21 without)
      const int dt_shift = 3 - __builtin_ctz(g.ng_v);          // log2 of the d-tiles per value group
#pragma unroll
      for (int dt = 0; dt < 8; ++dt)                           // (all eight tiles with their registers named at compile
        if (dt >> dt_shift == gcs) {                               // time; the stores of the other groups' tiles are skipped)
          float* dst = &sm_o[wave][h][16 * dt + 4 * L.j];
#pragma unroll
          for (int rr = 0; rr < 4; ++rr) dst[rr] = fmaf(st.acc[dt][rr], kInvUnitV, z);
        }
    }
  }
  // (records of kernels that carry their weights times different powers of two meet in one merge when channel-wise keys
  // add the residual tail: the difference to 2^10 goes into the record's maximum)
  if (grp == 0 && L.j == 0 && !upper) { sm_m[wave][h] = st.m + (10.0f - p_shift<BV>()); sm_l[wave][h] = l; }
  if constexpr (KSEQ) {
    if (32 * wave < n_old) {                       // (uniform: at most 4 wavefronts)
      const int64_t at = (int64_t)bh * g.resid * (2 * kHeadDim);
      const uint8_t* kb = reinterpret_cast<const uint8_t*>(cache.k_resid) + at;
      const uint8_t* vb = reinterpret_cast<const uint8_t*>(cache.v_resid) + at;
      const float kp = softmax_scale * kLog2e;
      if (g.raw_dtype == KVQ_BF16) buffer_step<R, true>(kb, vb, qbase, r_act, n_old, wave, L, kp, sm_buf[wave], sm_bufm[wave], sm_bufl[wave]);
      else buffer_step<R, false>(kb, vb, qbase, r_act, n_old, wave, L, kp, sm_buf[wave], sm_bufm[wave], sm_bufl[wave]);
    }
  }
  __syncthreads();

  // (the ring's last loads, which nothing reads, have come back: said here, or the compiler waits where their registers are used
  // again, inside the loop below, whose second turn -- more than 4 heads -- would then wait for the first one's record
  // stores: 10.73 us instead of 10.44 for 1500 tokens of 8 x 8 heads)
  __builtin_amdgcn_s_waitcnt(0x0F70);                // vmcnt(0)
  // the counter of this (batch, kv head)'s records (kvq_merge_count.h); the maximum is on its way while the wavefronts are merged
  MergeWord* const word = reinterpret_cast<MergeWord*>(ws + (int64_t)g.batch * q_heads * a.rec_splits * kRec) + bh;
  if (a.merge_tag != 0 && tid == 0 && n_rec > 1)
    (void)__hip_atomic_fetch_max(word, a.merge_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // ---- merge the wavefronts; write a partial record, or the result when there is one split
  // (plain exponentials here and in the merges below: a weight under 2^-126 comes out as 0, far under a binary32 rounding of any sum it enters)
  for (int idx = tid; idx < R * kHeadDim; idx += 64 * NW) {
    const int hh = idx / kHeadDim, d = idx % kHeadDim;
    float M = sm_m[0][hh];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, sm_m[w][hh]);
    if (do_append) M = fmaxf(M, sm_mnew[hh]);
    const int buf_recs = KSEQ ? (n_old + 31) >> 5 : 0;
    if constexpr (KSEQ)
      for (int w = 0; w < buf_recs; ++w) M = fmaxf(M, sm_bufm[w][hh]);
    float o = 0.f, ll = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(sm_m[w][hh] - M);
      o = fmaf(f, sm_o[w][hh][d], o);
      ll = fmaf(f, sm_l[w][hh], ll);
    }
    if (do_append) {                               // the new token: one weight of 1 (records carry their sums times 2^10)
      const float f = 1024.0f * __builtin_amdgcn_exp2f(sm_mnew[hh] - M);
      o = fmaf(f, sm_hat[1][d], o);
      ll += f;
    }
    if constexpr (KSEQ)
      for (int w = 0; w < buf_recs; ++w) {
        const float f = __builtin_amdgcn_exp2f(sm_bufm[w][hh] - M);
        o = fmaf(f, sm_buf[w][hh][d], o);
        ll = fmaf(f, sm_bufl[w][hh], ll);
      }
    if (hh >= r_act) continue;
    const int64_t hq = (int64_t)b * q_heads + hk * r_act + hh;
    if (a.extra_splits != 0) {
      // one more record per head lies in the workspace, written by an earlier launch on the same stream (the flushed
      // part of a cache with a residual buffer, when this launch is the buffer's): it joins here, and no merge launch
      // follows
      const float* er = ws + hq * a.extra_splits * kRec;
      const float me = er[kHeadDim], le = er[kHeadDim + 1], oe = er[d];
      const float Mn = fmaxf(M, me);
      const float f0 = __builtin_amdgcn_exp2f(M - Mn), fe = __builtin_amdgcn_exp2f(me - Mn);
      o = fmaf(fe, oe, o * f0);
      ll = fmaf(fe, le, ll * f0);
    }
    if (n_rec == 1) {
      const float val = o / ll;
      if (g.rotate_v) { sm_o[0][hh][d] = val; continue; }      // (only this thread touches element (hh, d))
      store_out(out, out_dtype, hq * kHeadDim + d, val);
    } else {
      // (device-scope stores: the record is read by a workgroup on another part of the chip, whose nearest cache is
      // not this one)
      float* rec = ws + (a.balance ? ((int64_t)slot * g.kv_heads + hk) * r_act + hh : hq * a.rec_splits + a.rec_base + split) * kRec;
      store_device(rec + d, o);
      if (d == 0) { store_device(rec + kHeadDim, M); store_device(rec + kHeadDim + 1, ll); }
    }
  }
  bool wrote_rows = n_rec == 1;               // this workgroup has left normalized rows (rotated values: in sm_o)
  if (a.merge_tag != 0 && n_rec > 1) {               // uniform: the launch's workgroups merge their records themselves
    // The workgroup of a (batch, kv head) that finishes last combines its records.  Every workgroup counts itself in, after
    // its record stores have been performed; the one that brings the count to n_rec reads all records back.  Nobody waits for
    // anybody.  The counter and its rules: kvq_merge_count.h.
    // Records and counter are device-scope atomic accesses, which go past the caches that are private to a part of the
    // chip; a device-scope FENCE is not used on purpose: it writes back and invalidates the whole second-level cache of the
    // workgroup's part of the chip, under the streaming loads of every other workgroup there, and was measured to cost the
    // 8B-layer step 10 us.  The order is carried by the wait below: a store is acknowledged when it has been performed, and a
    // barrier alone does not wait for it.
    __shared__ int sm_last;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");     // (costs nothing: keeps the compiler from moving a store behind the wait)
    __builtin_amdgcn_s_waitcnt(0x0F70);              // vmcnt(0): this wavefront's record stores are performed
    __syncthreads();                                 // (and so are the other wavefronts')
    if (tid == 0) {
      MergeWord before = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (merge_unmarked(before, a.merge_tag)) {     // (rare; a swap fails only because another workgroup got on)
        MergeWord seen = before + 1;
        while (merge_unmarked(seen, a.merge_tag) &&
               !__hip_atomic_compare_exchange_strong(word, &seen, a.merge_tag | 1ull, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {}
        before = merge_unmarked(seen, a.merge_tag) ? a.merge_tag
                                                   : __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      const bool last = merge_last(before, n_rec);
      if (last) __hip_atomic_store(word, a.merge_tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      sm_last = last;
    }
    __syncthreads();
    if (sm_last) {                                   // uniform over the workgroup
      // records of this (batch, kv head): the first one's place and the distance to the next, in records
      const int64_t rec0 = a.balance ? ((int64_t)slot0 * g.kv_heads + hk) * r_act : ((int64_t)b * q_heads + hk * r_act) * n_rec;
      const int64_t rec_step = a.balance ? q_heads : 1, head_step = a.balance ? 1 : n_rec;
      for (int idx = tid; idx < r_act * kHeadDim; idx += 64 * NW) {
        const int hh = idx / kHeadDim, d = idx % kHeadDim;
        const int64_t hq = (int64_t)b * q_heads + hk * r_act + hh;
        const float* rec = ws + (rec0 + hh * head_step) * kRec;
        // four records at a time, all 12 loads of a round in flight together (a record's maximum and sum are the same
        // words for the 128 threads of a head); rounds are chained by a running maximum as in the main loop
        float M = kNegBig, o = 0.f, ll = 0.f;
        if (n_rec == 2) {                            // (uniform; the usual number)
          const float* r1 = rec + rec_step * kRec;
          const float m0 = load_device(rec + kHeadDim), l0 = load_device(rec + kHeadDim + 1), o0 = load_device(rec + d);
          const float m1 = load_device(r1 + kHeadDim), l1 = load_device(r1 + kHeadDim + 1), o1 = load_device(r1 + d);
          M = fmaxf(m0, m1);
          const float f0 = __builtin_amdgcn_exp2f(m0 - M), f1 = __builtin_amdgcn_exp2f(m1 - M);
          o = fmaf(f1, o1, f0 * o0); ll = fmaf(f1, l1, f0 * l0);
        } else for (int s0 = 0; s0 < n_rec; s0 += 4) {
          float ms[4], ls[4], os[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float* r2 = rec + min(s0 + j, n_rec - 1) * rec_step * kRec;
            ms[j] = load_device(r2 + kHeadDim); ls[j] = load_device(r2 + kHeadDim + 1); os[j] = load_device(r2 + d);
          }
          float Mc = M;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (s0 + j >= n_rec) { ms[j] = kNegBig; ls[j] = 0.f; os[j] = 0.f; }
            Mc = fmaxf(Mc, ms[j]);
          }
          const float fo = __builtin_amdgcn_exp2f(M - Mc);
          o *= fo; ll *= fo;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float f = __builtin_amdgcn_exp2f(ms[j] - Mc);
            o = fmaf(f, os[j], o);
            ll = fmaf(f, ls[j], ll);
          }
          M = Mc;
        }
        const float val = o / ll;
        if (g.rotate_v) sm_o[0][hh][d] = val;
        else store_out(out, out_dtype, hq * kHeadDim + d, val);
      }
      wrote_rows = true;
    }
  }
  if (wrote_rows && g.rotate_v) {                    // uniform over the workgroup
    __syncthreads();
    if (tid < R * 16 && (tid >> 4) < r_act)
      store_unrotated_row(&sm_o[0][tid >> 4][0], tid & 15, g.signs_v, out, out_dtype,
                          (int64_t)b * q_heads + hk * r_act + (tid >> 4));
  }
}

// Combine the split records of one (b, hq): log-sum-exp merge, then normalize (and take rotated values back).
// 512 threads: four groups of 128 channels, group k takes the records s = k, k+4, ..., eight at a time with all their loads
// (maximum, sum, element) in flight together, under a running maximum of its own; one step through LDS adds the groups.  So
// up to 32 records cost one memory latency, which is what bounds the kernel (with a pass over the maxima in front of the sums
// it had two: whole steps, K4V2, before and now, 8 heads x 131071 tokens, 32 records, 27.1 and 26.6 us, x 8192, 16 records,
// 12.0 and 11.2; 2 x 8 x 8 heads x 16384 tokens, 16 records, 15.5 and 14.7; 4 x 7 heads x 131071, 64 records, 20.05 and 19.85).
struct RotV { int32_t on; uint32_t signs[4]; };
constexpr int kMergeGroups = 4, kMergeDeep = 8;
__global__ __launch_bounds__(128 * kMergeGroups) void merge_kernel(const float* __restrict__ ws, void* __restrict__ out,
                                                                   int out_dtype, int32_t n_splits, RotV rot) {
  __shared__ float row[kHeadDim];
  __shared__ float s_o[kMergeGroups][kHeadDim], s_m[kMergeGroups], s_l[kMergeGroups];
  const int64_t hq = blockIdx.x;
  const int tid = threadIdx.x, d = tid & (kHeadDim - 1), grp = tid >> 7;
  const float* rec = ws + hq * n_splits * kRec;
  float M = kNegBig, o = 0.f, l = 0.f;
  for (int s0 = grp; s0 < n_splits; s0 += kMergeGroups * kMergeDeep) {
    float ms[kMergeDeep], ls[kMergeDeep], os[kMergeDeep];
#pragma unroll
    for (int j = 0; j < kMergeDeep; ++j) {         // (past the last record its cache lines once more, cleared below)
      const float* r = rec + min(s0 + kMergeGroups * j, n_splits - 1) * kRec;
      ms[j] = r[kHeadDim]; ls[j] = r[kHeadDim + 1]; os[j] = r[d];
    }
    float Mc = M;
#pragma unroll
    for (int j = 0; j < kMergeDeep; ++j) {         // (cleared, not weighted by 0: an infinite value of an unquantized cache stays one)
      if (s0 + kMergeGroups * j >= n_splits) { ms[j] = kNegBig; ls[j] = 0.f; os[j] = 0.f; }
      Mc = fmaxf(Mc, ms[j]);
    }
    const float fo = __builtin_amdgcn_exp2f(M - Mc);
    o *= fo; l *= fo;
#pragma unroll
    for (int j = 0; j < kMergeDeep; ++j) {
      const float f = __builtin_amdgcn_exp2f(ms[j] - Mc);
      o = fmaf(f, os[j], o);
      l = fmaf(f, ls[j], l);
    }
    M = Mc;
  }
  s_o[grp][d] = o;
  if (d == 0) { s_m[grp] = M; s_l[grp] = l; }
  __syncthreads();
  if (grp != 0) {
    if (!rot.on) return;
  } else {
    M = s_m[0];
#pragma unroll
    for (int k = 1; k < kMergeGroups; ++k) M = fmaxf(M, s_m[k]);
    o = 0.f; l = 0.f;
#pragma unroll
    for (int k = 0; k < kMergeGroups; ++k) {
      const float f = __builtin_amdgcn_exp2f(s_m[k] - M);
      o = fmaf(f, s_o[k][d], o);
      l = fmaf(f, s_l[k], l);
    }
  }
  const float val = o / l;
  if (rot.on) {                                      // uniform
    if (grp == 0) row[d] = val;
    __syncthreads();
    if (tid < 16) store_unrotated_row(row, tid, rot.signs, out, out_dtype, hq);
    return;
  }
  store_out(out, out_dtype, hq * kHeadDim + d, val);
}

inline RotV rot_v_of(const Geom& g) {
  RotV r{g.rotate_v, {g.signs_v[0], g.signs_v[1], g.signs_v[2], g.signs_v[3]}};
  return r;
}

// The same merge for up to 8 records (5 to 8 splits, 3 to 8 for attention alone over 7 or 8 heads, and those of token-wise keys behind a
// residual buffer, which come from two launches): one wavefront pair per head, every
// record's maximum, sum and element loaded at once -- 24 independent loads, one memory latency -- and no step through
// LDS.
constexpr int kMergeFew = 8;
__global__ __launch_bounds__(kHeadDim) void merge_few_kernel(const float* __restrict__ ws, void* __restrict__ out,
                                                             int out_dtype, int32_t n_splits, RotV rot) {
  __shared__ float row[kHeadDim];
  const int64_t hq = blockIdx.x;
  const int d = threadIdx.x;
  const float* rec = ws + hq * n_splits * kRec;
  float m[kMergeFew], l[kMergeFew], o[kMergeFew];
#pragma unroll
  for (int j = 0; j < kMergeFew; ++j) {
    const float* r = rec + min(j, n_splits - 1) * kRec;       // (past the last record its cache lines once more, cleared below)
    m[j] = r[kHeadDim]; l[j] = r[kHeadDim + 1]; o[j] = r[d];
  }
  float M = m[0];
#pragma unroll
  for (int j = 1; j < kMergeFew; ++j) {
    if (j >= n_splits) { m[j] = kNegBig; l[j] = 0.f; o[j] = 0.f; }
    M = fmaxf(M, m[j]);
  }
  float os = 0.f, ls = 0.f;
#pragma unroll
  for (int j = 0; j < kMergeFew; ++j) {
    const float f = __builtin_amdgcn_exp2f(m[j] - M);
    os = fmaf(f, o[j], os);
    ls = fmaf(f, l[j], ls);
  }
  const float val = os / ls;
  if (rot.on) {                                      // uniform
    row[d] = val;
    __syncthreads();
    if (d < 16) store_unrotated_row(row, d, rot.signs, out, out_dtype, hq);
    return;
  }
  store_out(out, out_dtype, hq * kHeadDim + d, val);
}

// Merge `records` partial records per (batch, query head) into the output.
inline void launch_merge(const float* ws, void* out, int out_dtype, int32_t heads, int32_t records, RotV rot, hipStream_t stream) {
  if (records <= kMergeFew)
    hipLaunchKernelGGL(merge_few_kernel, dim3(heads), dim3(kHeadDim), 0, stream, ws, out, out_dtype, records, rot);
  else
    hipLaunchKernelGGL(merge_kernel, dim3(heads), dim3(128 * kMergeGroups), 0, stream, ws, out, out_dtype, records, rot);
}


template <int BK, int BV, int R, bool BF, int NCK, int NCV, bool KSEQ, bool PAGED, bool HALF = false>
void launch_nw(const DecodeArgs& a, const DecodePlan& plan, dim3 grid, hipStream_t stream) {
  if constexpr (BK != 16 && BV != 16 && !KSEQ) {
    if (a.g.rotate_v) {
      if (plan.waves_per_wg == 8)
        hipLaunchKernelGGL((decode_kernel<BK, BV, R, 8, BF, NCK, NCV, KSEQ, PAGED, true, HALF>), grid, dim3(512), 0, stream, a);
      else
        hipLaunchKernelGGL((decode_kernel<BK, BV, R, 4, BF, NCK, NCV, KSEQ, PAGED, true, HALF>), grid, dim3(256), 0, stream, a);
      return;
    }
  }
  if (plan.waves_per_wg == 8)
    hipLaunchKernelGGL((decode_kernel<BK, BV, R, 8, BF, NCK, NCV, KSEQ, PAGED, false, HALF>), grid, dim3(512), 0, stream, a);
  else
    hipLaunchKernelGGL((decode_kernel<BK, BV, R, 4, BF, NCK, NCV, KSEQ, PAGED, false, HALF>), grid, dim3(256), 0, stream, a);
}

// One column set: at most 8 columns on either side take two tiles side by side (channel-wise keys: two columns a head).  Always
// so up to two heads, never for channel-wise keys of 8; unquantized tensors, whose step is bound by its bytes, keep one tile after the other.
template <int BK, int BV, int R, bool BF, bool KSEQ, bool PAGED>
void launch_columns(const DecodeArgs& a, const DecodePlan& plan, dim3 grid, hipStream_t stream) {
  constexpr bool kMay = BK != 16 && BV != 16 && !(KSEQ && R == 8), kMust = kMay && R <= 2;
  if constexpr (kMust) {
    launch_nw<BK, BV, R, BF, 1, 1, KSEQ, PAGED, true>(a, plan, grid, stream);
  } else {
    if constexpr (kMay) {
      if (R * (KSEQ ? 2 : a.g.ng_k) <= 8 && R * a.g.ng_v <= 8) {
        launch_nw<BK, BV, R, BF, 1, 1, KSEQ, PAGED, true>(a, plan, grid, stream);
        return;
      }
    }
    launch_nw<BK, BV, R, BF, 1, 1, KSEQ, PAGED>(a, plan, grid, stream);
  }
}

// column sets: two only where 8 heads meet four groups (32 columns); quantized caches only
template <int BK, int BV, int R, bool BF, bool KSEQ, bool PAGED>
hipError_t launch_sets(const DecodeArgs& a, const DecodePlan& plan, dim3 grid, hipStream_t stream) {
  const bool k2 = R * a.g.ng_k > 16, v2 = R * a.g.ng_v > 16;
  if constexpr (R == 8 && BK != 16 && BV != 16) {
    if constexpr (KSEQ) {
      if (k2) return hipErrorInvalidValue;
      if (v2) launch_nw<BK, BV, R, BF, 1, 2, true, PAGED>(a, plan, grid, stream);
      else launch_columns<BK, BV, R, BF, true, PAGED>(a, plan, grid, stream);
    } else {
      if (k2 && v2) launch_nw<BK, BV, R, BF, 2, 2, false, PAGED>(a, plan, grid, stream);
      else if (k2) launch_nw<BK, BV, R, BF, 2, 1, false, PAGED>(a, plan, grid, stream);
      else if (v2) launch_nw<BK, BV, R, BF, 1, 2, false, PAGED>(a, plan, grid, stream);
      else launch_columns<BK, BV, R, BF, false, PAGED>(a, plan, grid, stream);
    }
  } else {
    if (k2 || v2) return hipErrorInvalidValue;
    launch_columns<BK, BV, R, BF, KSEQ, PAGED>(a, plan, grid, stream);
  }
  return hipGetLastError();
}

template <int BK, int BV, int R, bool BF = false, bool KSEQ = false>
hipError_t launch_one(const DecodeArgs& a, const DecodePlan& plan, hipStream_t stream) {
  const dim3 grid = a.balance ? dim3(1, a.g.kv_heads, a.balance) : dim3(plan.n_splits, a.g.kv_heads, a.g.batch);
  hipError_t e;
  e = a.g.page_shift ? launch_sets<BK, BV, R, BF, KSEQ, true>(a, plan, grid, stream)
                     : launch_sets<BK, BV, R, BF, KSEQ, false>(a, plan, grid, stream);
  // the records of this launch are all there is: merge them, in the launch itself where that pays (merge_tag), else
  // here (otherwise the caller adds launches and merges)
  if (e != hipSuccess || a.rec_splits == 1 || a.rec_splits != plan.n_splits || a.merge_tag != 0) return e;
  launch_merge(a.ws, a.out, a.out_dtype, a.g.batch * a.q_heads, a.rec_splits, rot_v_of(a.g), stream);
  return hipGetLastError();
}

template <int BK, int BV, bool BF = false, bool KSEQ = false>
hipError_t launch_r(int R, const DecodeArgs& a, const DecodePlan& plan, hipStream_t stream) {
  switch (R) {
    case 1: return launch_one<BK, BV, 1, BF, KSEQ>(a, plan, stream);
    case 2: return launch_one<BK, BV, 2, BF, KSEQ>(a, plan, stream);
    case 4: return launch_one<BK, BV, 4, BF, KSEQ>(a, plan, stream);
    case 8: return launch_one<BK, BV, 8, BF, KSEQ>(a, plan, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace

#define KVQ_CAT2(a, b, c) a##b##_##c
#define KVQ_CAT(a, b, c) KVQ_CAT2(a, b, c)

#if defined(KVQ_INST_BK)
// ---- instance translation unit: the kernels of one (b_K, b_V) pair behind one launcher -------------------------------
hipError_t KVQ_CAT(launch_decode_inst_, KVQ_INST_BK, KVQ_INST_BV)(int R, const DecodeArgs& a, const DecodePlan& plan,
                                                                  hipStream_t stream) {
#if KVQ_INST_BK == 16 || KVQ_INST_BV == 16
  // one tensor or both unquantized: token-wise kernels only, typed by the 16-bit patterns' type
  return a.g.raw_dtype == KVQ_BF16 ? launch_r<KVQ_INST_BK, KVQ_INST_BV, true>(R, a, plan, stream)
                                   : launch_r<KVQ_INST_BK, KVQ_INST_BV, false>(R, a, plan, stream);
#else
  if (a.g.axis_k == KVQ_AXIS_SEQ) return launch_r<KVQ_INST_BK, KVQ_INST_BV, false, true>(R, a, plan, stream);
  return launch_r<KVQ_INST_BK, KVQ_INST_BV>(R, a, plan, stream);
#endif
}

#else
// ---- dispatcher translation unit ----------------------------------------------------------------------------------------
#ifndef KVQ_FOR_EACH_PAIR      // (a development build may name fewer pairs on the command line)
#define KVQ_FOR_EACH_PAIR(X) X(4, 2) X(2, 4) X(4, 4) X(8, 8) X(2, 2) X(8, 4) X(8, 2) X(4, 8) X(2, 8) X(16, 16) \
  X(3, 2) X(3, 4) X(3, 8) X(6, 2) X(6, 4) X(6, 8) X(1, 2) X(1, 4) X(1, 8) \
  X(1, 1) X(2, 1) X(3, 1) X(4, 1) X(6, 1) X(8, 1) \
  X(1, 3) X(2, 3) X(3, 3) X(4, 3) X(6, 3) X(8, 3) X(1, 6) X(2, 6) X(3, 6) X(4, 6) X(6, 6) X(8, 6) \
  X(16, 1) X(16, 2) X(16, 3) X(16, 4) X(16, 6) X(16, 8) X(1, 16) X(2, 16) X(3, 16) X(4, 16) X(6, 16) X(8, 16)
#endif
#define KVQ_DECL(BK_, BV_) \
  hipError_t KVQ_CAT(launch_decode_inst_, BK_, BV_)(int R, const DecodeArgs& a, const DecodePlan& plan, hipStream_t stream);
KVQ_FOR_EACH_PAIR(KVQ_DECL)
#undef KVQ_DECL

// Columns are laid out for a power-of-two number of heads per KV head.
int padded_heads(int r) { return r <= 1 ? 1 : r <= 2 ? 2 : r <= 4 ? 4 : 8; }

bool decode_supported(const Geom& g, int32_t q_heads) {
  const int r = q_heads / g.kv_heads;
  if (r < 1 || r > 8) return false;
  const int R = padded_heads(r);
  if (R * g.ng_k > 32 || R * g.ng_v > 32) return false;        // head x group columns: at most two 16-wide tiles
  if ((g.bits_k == 16) != (g.bits_v == 16)) {                  // one tensor unquantized, the other not:
    if (R * g.ng_k > 16 || R * g.ng_v > 16) return false;      // one column set, token-wise keys, values not rotated
    if (g.axis_k == KVQ_AXIS_SEQ || g.resid || g.rotate_v) return false;
  }
  return true;
}

// Compute units of the current device, asked once per device (a partitioned or binned part has fewer than the 256 of
// a whole MI355X).  Without a usable device (the host-only size queries on a machine with no GPU) the whole part's count.
int device_compute_units() {
  constexpr int kFull = 256, kMaxDevices = 64;
  static std::atomic<int> cached[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return kFull; }
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      n = kFull;
    }
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

namespace {
// Wavefronts per (b, h_kv) stream that fill the chip once, and what a sequence of n_steps steps can use of them.  A few workgroups more
// than the chip takes at a time cost a whole round, so the plan rounds the wavefronts per stream down; the bound on the
// records, which callers have sized workspaces by, rounds up as the plan once did.  Rounded up and down, K4V2: 11 x 8 heads x 6000
// tokens (88 streams in 3 and 2 parts) 21.5 and 14.4 us, x 16000 43.0 and 29.1; 17 x 8 x 6000 (2 parts and 1) 28.5 and 20.6; 33 x 8
// (one workgroup of 8 wavefronts and of 4, two of which share a unit) x 700 11.7 and 9.3, x 6000 45.0 and 38.4.
// Two wavefronts per SIMD are counted for every instance.  Token-wise K4V2 of one column set needs 144 to 167 registers, which leave room for a
// third (channel-wise and two-set ones mostly need more); no plan by three has been measured.
struct WaveBudget { int waves, nw, splits; };
WaveBudget wave_budget(const Geom& g, int n_steps, bool bound) {
  const int streams = g.batch * g.kv_heads;
  const int total_waves = device_compute_units() * 4 * KVQ_WAVES_PER_SIMD;
  int waves_per_stream = (total_waves + (bound ? streams - 1 : 0)) / streams;
  // at least two steps per wavefront (four or eight, i.e. fewer splits and at B=8, T=2048 the two-record merge inside
  // the launch instead of the merge launch, measure 13.7 and 14.6 us there against 11.9)
  const int max_waves = (n_steps + 1) / 2;
  if (waves_per_stream > max_waves) waves_per_stream = max_waves;
  if (waves_per_stream < 4) waves_per_stream = 4;
  const int nw = waves_per_stream >= 8 ? 8 : 4;
  int splits = waves_per_stream / nw;
  if (splits < 1) splits = 1;
  return WaveBudget{waves_per_stream, nw, splits};
}
int plan_steps(const Geom& g, int32_t seq_len) {
  return g.resid ? seq_len / g.resid * (g.resid / 32) : (seq_len + 31) / 32;      // (a residual buffer: the flushed tokens only)
}
}  // namespace

namespace {
// The plan for every layout: fill the chip exactly once, at least two steps per wavefront.
DecodePlan plan_coarse(const Geom& g, int32_t seq_len) {
  // Fill the chip exactly once: compute units x 4 SIMDs x KVQ_WAVES_PER_SIMD wavefronts, spread over the (b,h) streams.
  // Workgroups of 8 wavefronts halve the number of sequence splits (none at all from 256 streams up, where the
  // merge kernel and the workspace traffic disappear); each wavefront should still own a few steps.
  // Channel-wise keys: the plan covers the flushed tokens only (whole 64-token blocks, two steps each, taken in pairs);
  // n_splits = 0 when nothing is flushed yet.  The tokens in the buffer come with the last split (token-wise keys behind a buffer, and
  // nothing flushed yet: a launch of their own).
  const int unit = g.axis_k == KVQ_AXIS_SEQ ? 2 : 1;
  const int n_steps = plan_steps(g, seq_len);
  if (n_steps == 0) return DecodePlan{0, 0, 4};
  const WaveBudget wb = wave_budget(g, n_steps, false);
  const int nw = wb.nw;
  int sps = (n_steps + wb.splits - 1) / wb.splits;
  sps = (sps + nw * unit - 1) / (nw * unit) * (nw * unit);
  const int splits = (n_steps + sps - 1) / sps;
  return DecodePlan{splits, sps, nw};
}

// Sequences without a residual buffer (whose plan takes whole blocks as it is) are cut with their parts' size in view.  n8: steps per
// wavefront if one workgroup of 8 took the sequence; most: workgroups per sequence that fill the chip.
//   - n8 <= 3: one workgroup and nothing to merge.
//   - n8 == 4: four parts of one step per wavefront, which the launch merges itself, where the chip has room for them and there are up to 4
//     heads to merge (more: one part up to 30 steps, then two).
//   - above that up to 8 parts of two or three steps per wavefront.  Up to 4 heads leave this to the coarse plan: a few parts more, and with
//     them the second launch, gain 0.5 us on the device and lose 1 where the host paces.
//   - where more than three steps per wavefront are left, as few as all the parts allow: from 9 records on a larger merge launch costs a
//     microsecond more.
// The lines were drawn on K4V2.  Wider rows, captured in a graph, against the coarse plan: with more than four heads and in long sequences within 1 %
// (K8V8, 8 to 352 sequences, 500 to 16384 tokens; unquantized rows: below); unquantized sequences of 40 and 100 tokens would take four wavefronts 2 to 6 %
// faster (8 x 8 heads x 100, 8 query heads, 6.35 and 6.69 us, 4 query heads 5.46 and 5.56), K8V8 and unquantized ones of 300 tokens and one query
// head too (8 x 8 heads 6.34 and 6.49, 7.50 and 7.68).
// Fused steps, K4V2, 4 query heads unless said, before (the coarse plan) and so, captured in a graph: 8 heads x 800 tokens 7.07 and 6.44 us,
// x 1024 7.43 and 6.85 (1 query head 7.38 and 6.84), x 7000 10.73 and 9.93, x 8192 10.12 and 9.28, x 10000 11.12 and 10.51; 8 x 8
// heads x 1024 8.23 and 7.90; 4 x 8 heads x 3000, 8 query heads, back to back 10.32 and 9.45.  On the other side of the lines: 8 heads x 640 tokens in
// one part 6.49, in three 6.94; 8 heads x 800, 8 query heads, in one part 8.01, in four 8.12; 16 x 8 heads x 800 in one part 7.89, in two
// 8.10; 8 heads x 3000 in 4 parts 8.93, back to back 8.52, in 6 parts 8.45 and 9.57; 8 heads x 4096 in 8 parts 8.49, in 16 9.53, x
// 6000 in 8 parts 9.12, in 24 9.73; x 8192 in 8 parts 10.46, in 16 10.17, in 32 9.28.
struct FinePlan { int splits, steps; };            // steps per wavefront; splits = 0: the coarse plan
// Rows of 512 bytes (wide: both tensors unquantized; K8V8 takes half) are the other way round: one step of eight wavefronts is 128 KB, so the parts
// are as many as fill the chip down to one step per wavefront, from 14 steps on (13: 8 query heads, 8 x 8 heads 11.5 and 10.4 us, 2 x 8 9.1 and 9.3).  Attention, with the lines above and so: 2 x 8 heads x 700 tokens, 4 query
// heads, 12.4 and 8.8 us; 17 x 4 heads x 907, 7 query heads, 18.0 and 15.0, x 500 12.3 and 10.4; 4 x 8 x 2000 14.1 and 10.9; K8V8 2 x 8 x 700 8.6 and 7.8.
// Where the chip has room for two parts, 17 to 20 steps (more than 4 heads: to 22) stay in one: one part per step of a wavefront would be three, and
// of two parts of two steps the second would get 1 to 4 steps of 8 wavefronts.  In two parts and in one, 16 x 8 heads, 17, 18, 20, 21 and 24
// steps, 8 query heads, 13.5 to 6.0 % slower up to 21 and 1.8 % faster at 24; 4 query heads 12.0, 8.0, 3.6, 1.1 % slower and 2.4 % faster; 11 x 8, 4
// query heads, 10.5, 8.0, 1.6 % slower, 2.4 and 7.3 % faster (16 x 8 x 573 tokens, 8 query heads, 15.5 and 14.3 us).
FinePlan fine_plan(int n_steps, int most, int heads, bool wide) {
  const int n8 = (n_steps + 7) / 8;
  if (wide && most > 1 && n_steps >= 14 && !(most == 2 && n_steps > 16 && n_steps <= (heads > 4 ? 22 : 20))) {
    const int steps = (n8 + most - 1) / most;
    return FinePlan{(n8 + steps - 1) / steps, steps};
  }
  if (n8 == 4 && most >= 4 && heads <= 4) return FinePlan{4, 1};
  if (most <= 1 || n8 <= 3 || n_steps < 31) return FinePlan{1, n8};
  const int few = most < 8 ? most : 8;
  int steps;
  if (n8 <= 3 * few) {
    if (heads <= 4) return FinePlan{0, 0};
    steps = (n8 + few - 1) / few;
    if (steps < 2) steps = 2;
  } else {
    steps = (n8 + most - 1) / most;
  }
  return FinePlan{(n8 + steps - 1) / steps, steps};
}
// No length up to n_steps takes more parts.
int fine_bound(int n_steps, int most, bool wide) {
  const int n8 = (n_steps + 7) / 8;
  if (wide) return most <= 1 || n_steps < 14 ? 1 : n8 < most ? n8 : most;
  if (most <= 1 || n8 <= 3) return 1;
  const int few = most < 8 ? most : 8, two = (n8 + 1) / 2 > 4 ? (n8 + 1) / 2 : 4;
  if (n8 <= 3 * few) return two < few ? two : few;
  return n8 < most ? n8 : most;
}
bool wide_rows(const Geom& g) { return g.bits_k == 16 && g.bits_v == 16; }
// Workgroups of 8 wavefronts per sequence that fill the chip; 0 where there are too many sequences for one each.
int fine_most(const Geom& g, bool bound) {
  const int streams = g.batch * g.kv_heads, waves = device_compute_units() * 4 * KVQ_WAVES_PER_SIMD;
  return g.resid ? 0 : (waves + (bound ? streams - 1 : 0)) / streams / 8;
}
}  // namespace

// Sequences of different lengths: a launch may deal its workgroups of nw wavefronts out by the lengths (balanced_share).  How many: as
// many as fill the chip, where the plan takes more than half of it; sequences of one part each, 129 to 255 and 257 to 511 streams, leave
// some over for the longest.  Where the plan takes less (few, short sequences), its own number.
// Which plans: two parts of at least 6 steps per wavefront (wide rows: in proportion to their width, 4 at least), more of at least 12 (with
// eight it loses, 4 sequences up to 8000 tokens: 14.4 us against 12.3), sequences of one part from deal_line1 on.  With less, looking at all the
// lengths first outweighs it.  Two parts of wide rows, nothing dealt out and so, lengths even from a share of the longest up to it: K8V8, 11 x 8
// heads x 2200 tokens, 4 query heads, from 0.03 on 15.4 and 11.9 us, from 0.2 on 15.7 and 12.9, from 0.8 on 16.9 and 16.7; of three steps per
// wavefront, 16 x 8 x 1300, 8 query heads, from 0.03 on 5 % faster and from 0.8 on 5 % slower.
namespace {
// The steps that a dealt-out part has to save to pay, and the lines, are drawn on rows of up to 8 bits (codes of key and value); a step of wider
// rows takes longer, in proportion (of four wavefronts deal_most has figures of its own).
int by_width(const Geom& g, int steps) { const int bits = g.bits_k + g.bits_v; return bits > 8 ? (8 * steps + bits - 1) / bits : steps; }
int deal_line1(const Geom& g, int nw) { return nw == 8 ? by_width(g, 72) : g.bits_k + g.bits_v > 8 ? 40 : 44; }
int deal_line2(const Geom& g, int nw) { return by_width(g, 6 * nw) > 4 * nw ? by_width(g, 6 * nw) : 4 * nw; }
bool deals(const Geom& g, const DecodePlan& p) {
  if (g.resid || g.batch < 2 || g.batch > 64 || p.n_splits < 1 || p.n_splits > 4) return false;
  return p.steps_per_split >= (p.n_splits == 1 ? deal_line1(g, p.waves_per_wg) : p.n_splits == 2 ? deal_line2(g, p.waves_per_wg) : 12 * p.waves_per_wg);
}
// The longest part that pays.  Sequences of one part have no records yet: the search, the records and their merge are 2 to 3 us, five steps of
// eight wavefronts (four of the shortest), and an eighth of the part at least, because the workgroups that come on top share the memory.  Of four wavefronts two workgroups
// share a unit: seven steps and 3/10 (nine and a quarter where there are more than 4 heads to merge), of wide rows four and 2/9 (six and a quarter),
// and nine to twelve steps always do.  Sequences of several parts merge in any case: two steps, and 3/16.
// One part, in turn with nothing dealt out, K4V2 and 4 query heads unless said, steps per wavefront planned and dealt out, lengths even from a share of the
// longest up to it.  Eight wavefronts: 17 x 8 heads x 3500 tokens, from 0.65 on, 14 -> 10: 15.2 us for 13.8, from 0.05 on, 14 -> 6: 11.7 for 13.7; 24 x 8 x 8000,
// 32 -> 28: 31.4 for 30.1, 32 -> 23: 26.1 for 27.0; 18 to 30 x 8, shares from 0.02 to 0.8, 36 -> 29 to 30 1 to 4 % faster (K2V2 2 to 6, K3V2 3 to 7), 36 -> 31 between 2 %
// slower and 4 % faster, 18 -> 13 0 to 5 %, 12 -> 7 5 to 13 %, 9 -> 4 1 to 10 %, 9 -> 5 3 to 10 %; four steps of more saved 4 % faster (K3V2) to 3 % slower (K4V4; 12 -> 8, 14 -> 10, 17 -> 13), three 2 % faster to 9 %
// slower; K8V8 gains from three steps on.
// Four wavefronts, 33 to 60 x 8 heads, shares from 0.03 to 0.7, means of up to 6 batches, per cent faster than nothing dealt out (-: slower).  The sequences
// in random order: in falling order of their lengths the planned parts share the units best, and it pays up to 15 less.  K4V2, 4 query heads: 11 -> 4 5, 11 -> 5 0,
// 15 -> 8 0, 15 -> 11 -8, 20 -> 12 1, 20 -> 14 -1, 25 -> 16 3, 25 -> 17 -1, 25 -> 18 -3, 25 -> 20 -8, 40 -> 31 -1, 71 -> 62 -2 (1 query head 2 to 5 better); 8 query heads: 11 -> 5
// -5, 15 -> 6 2, 15 -> 8 1, 20 -> 9 7, 20 -> 10 1, 20 -> 12 2, 20 -> 15 -8, 25 -> 14 13, 25 -> 16 2, 25 -> 18 -2, 40 -> 30 2, 40 -> 31 -3, 71 -> 50 7, 71 -> 59 4.  K8V8, 4 query
// heads: 11 -> 5 21, 11 -> 7 9, 15 -> 8 15, 15 -> 11 4, 20 -> 14 13, 20 -> 16 3, 25 -> 19 5, 25 -> 20 -4, 40 -> 31 5, 71 -> 62 2; 8 query heads: 11 -> 5 15, 11 -> 7 3, 15 -> 9 1, 15
// -> 11 -2, 20 -> 14 9, 20 -> 16 -2, 25 -> 18 7, 25 -> 20 -6, 40 -> 31 3, 71 -> 59 11, 71 -> 62 2.  Of eight steps planned the means are level or worse.
// Several parts, against the plan's own number dealt out: 11 x 8 x 3500, 7 -> 7: 12.8 for 11.6, 7 -> 6: 12.2; 7 x 8 x 16000, 16 -> 14: 21.8 for
// 21.0; 11 x 8 x 8000, 16 -> 9: 14.5 for 18.7.
int deal_most(const Geom& g, const DecodePlan& p, int heads) {
  const int nw = p.waves_per_wg, q = p.steps_per_split;
  const bool wide = g.bits_k + g.bits_v > 8;
  auto larger = [](int a, int b) { return a > b ? a : b; };
  auto smaller = [](int a, int b) { return a < b ? a : b; };
  int saved;
  if (p.n_splits > 1) saved = larger(by_width(g, 2 * nw), by_width(g, q * 3 / 16));
  else if (nw == 8) saved = larger(!wide && q <= 80 ? 32 : by_width(g, 40), by_width(g, q / 8));
  else if (wide) saved = heads > 4 ? larger(24, smaller(q / 4, 36)) : larger(16, smaller(q * 2 / 9, 36));
  else saved = heads > 4 ? larger(36, smaller(q / 4, 48)) : larger(28, smaller(q * 3 / 10, 40));
  return (q - saved) / nw * nw;
}
int full_slots(const Geom& g, int nw) { return device_compute_units() * 4 * KVQ_WAVES_PER_SIMD / nw / g.kv_heads; }
int deal_records(const Geom& g, int slots) { return (slots + g.batch - 1) / g.batch; }      // of the workspace, per (batch, kv head)
// No plan of more than half the chip in up to 4 parts a sequence, for lengths up to n_steps, takes more.  (A part is rounded up to whole
// wavefronts before it is held against the line, and so is the length here.)
int deal_bound(const Geom& g, int n_steps) {
  const int streams = g.batch * g.kv_heads, nw = streams <= device_compute_units() ? 8 : 4;
  const int line = deal_line1(g, nw) < deal_line2(g, nw) ? deal_line1(g, nw) : deal_line2(g, nw);
  if (g.resid || g.batch < 2 || g.batch > 64 || (n_steps + nw - 1) / nw * nw < line || 8 * streams <= device_compute_units()) return 1;
  const int records = deal_records(g, full_slots(g, nw));
  return records < 8 ? records : 8;
}
}  // namespace

// Upper bound, over every length up to seq_len, of the partial records per (batch, query head) that one decode call
// writes: one per split (token-wise keys behind a residual buffer: of the flushed blocks) plus, for token-wise keys behind a buffer, one
// for the tokens in it.  The number of splits
// before the steps are dealt out never shrinks as the sequence grows, and dealing them out in whole multiples of the
// workgroup's wavefronts only ever lowers it.  The workspace is sized for this bound, so a workspace sized once for the longest sequence serves every
// shorter one (the exact count is not monotone in the length).
// least: what a call must bring.  That is the coarse plan's records: with less than the full bound the call falls back on that plan.  And
// channel-wise keys, whose last split takes the buffer's tokens along, write none for them; the full bound counts one all the same,
// as it did when they did: the figure that callers ask for, and may have kept, does not change.
int32_t decode_records_bound(const Geom& g, int32_t seq_len, bool least) {
  const int n_steps = plan_steps(g, seq_len);
  if (n_steps == 0) return 1;
  const int splits = wave_budget(g, n_steps, true).splits;
  if (g.resid) return least && g.axis_k == KVQ_AXIS_SEQ ? splits : splits + 1;
  const int fine = least ? 0 : fine_bound(n_steps, fine_most(g, true), wide_rows(g));
  const int dealt = least ? 0 : deal_bound(g, n_steps);
  return dealt > fine && dealt > splits ? dealt : fine > splits ? fine : splits;
}

// heads: query heads per kv head; room: records per query head that the workspace holds.
static DecodePlan plan_parts(const Geom& g, int32_t seq_len, int heads, int64_t room) {
  const int n_steps = plan_steps(g, seq_len), most = n_steps ? fine_most(g, false) : 0;
  if (most < 1) return plan_coarse(g, seq_len);
  const FinePlan f = fine_plan(n_steps, most, heads, wide_rows(g));
  if (f.splits == 0 || (f.splits > 1 && f.splits > room)) return plan_coarse(g, seq_len);
  // (fewer than 8 steps and one or two heads: four wavefronts have less to merge.  7 steps, 4 and 8 wavefronts, 1 head 5.02 and 5.10 us,
  // 2 heads 5.10 and 5.20, 3 heads 5.56 and 5.14, 8 heads 6.62 and 6.23; 8 steps, 1 head 5.63 and 5.29, 8 heads 7.26 and 6.45)
  return DecodePlan{f.splits, 8 * f.steps, n_steps < 8 && heads < 3 ? 4 : 8};
}

DecodePlan plan_decode(const Geom& g, int32_t seq_len, int heads, int64_t room, bool ragged) {
  DecodePlan p = plan_parts(g, seq_len, heads, room);
  if (!ragged || !deals(g, p)) return p;
  p.deal_pays = deal_most(g, p, heads);
  const int own = p.n_splits * g.batch, full = full_slots(g, p.waves_per_wg);
  if (full > own && full < 2 * own && deal_records(g, full) <= room) p.slots = full;
  else if (p.n_splits > 1) p.slots = own;
  return p;
}

// Where the launch's own workgroups merge the records instead of a second launch.  Counting in, after the wait for the
// record stores, and reading the records back cost the last workgroup about what a dependent launch costs, and more the more
// it has to read (a workgroup's threads take more than 4 heads in two turns): up to four records, except that attention
// alone over 7 or 8 heads leaves three and four to the second launch.  Measured in turn, K4V2 and K4V4, 1 to 10 sequences of 2 to 8
// kv heads, 700 to 12000 tokens, the launch's own merge against the merge launch: three and four records of 1 head, attention,
// 2 to 10 % faster (4 x 8 heads x 2000 tokens 8.9 against 9.6 us), of 5 and 6 heads from 2.6 % faster to 2.3 % slower, of 7
// and 8 from 1 % faster to 4 % slower (4 x 8 x 8 heads x 2000 tokens 10.7 against 10.3); with the fused append, of 5 to 8
// heads, up to 3.5 % faster.  Five to eight records of 1 head from 2 % faster to 4 % slower, of 4 heads from 3 % faster to
// 5 % slower, of 8 heads 3 to 14 % slower (4 x 8 x 8 heads x 2500 tokens 11.8 against 10.4 us).
constexpr int kMergeHereMost = 4, kMergeHereMostAlone = 2, kAloneHeads = 6;
// The number such a launch carries (0: it does not merge): a greater one than all launches before it.  A replayed graph launch
// carries its number again.
static MergeWord next_merge_tag() {
  static std::atomic<MergeWord> launches{0};
  return merge_tag(launches.fetch_add(1, std::memory_order_relaxed));
}
static MergeWord merge_tag_for(int records, int most = kMergeHereMost) {
  return records >= 2 && records <= most ? next_merge_tag() : 0;
}

hipError_t launch_decode_attention(const Geom& g, const kvq_cache& c, const void* q, int q_dtype, int32_t q_heads,
                                   int32_t seq_len, float softmax_scale, void* out, int out_dtype, float* workspace,
                                   const DecodePlan& plan, const AppendOne* app, hipStream_t stream,
                                   const int32_t* seq_lens, int32_t lens_offset) {
  const int R = padded_heads(q_heads / g.kv_heads);
  DecodeArgs a{};
  a.heads_per_kv = q_heads / g.kv_heads;
  a.seq_lens = seq_lens; a.lens_offset = lens_offset;
  a.g = g; a.cache = c;
  a.q = (const uint16_t*)q; a.q_bf16 = q_dtype == KVQ_BF16 ? 1 : 0; a.q_heads = q_heads;
  a.seq_len = seq_len; a.softmax_scale = softmax_scale;
  a.ws = workspace; a.out = out; a.out_dtype = out_dtype;
  a.n_splits = plan.n_splits; a.steps_per_split = plan.steps_per_split;
  a.rec_splits = plan.n_splits; a.rec_base = 0;
  a.merge_tag = 0;
  if (g.resid) {
    // a residual buffer: flushed blocks from the codes (plan; channel-wise or token-wise keys), the newest tokens from
    // the buffer: by the same launch where the keys are channel-wise, else (and where nothing is flushed yet) by the unquantized
    // kernel, all partial records merged at the end
    // (per-sequence lengths: seq_len is their bound; every sequence's own flushed part and tail are cut out on the
    // device, the tail launch always runs, and a sequence without one of the parts gets empty records for it)
    const bool varlen = seq_lens != nullptr;
    const int32_t RL = g.resid;
    const int32_t n_flushed = seq_len / RL * RL;
    const int32_t tail = varlen ? (n_flushed ? RL - 1 : seq_len) : seq_len - n_flushed;
    if (g.axis_k == KVQ_AXIS_SEQ && n_flushed) {
      // channel-wise keys: the flushed blocks' launch takes the buffer's tokens along (buffer_step)
      a.seq_len = n_flushed; a.lens_mode = 1; a.lens_bound = seq_len; a.lens_block = RL;
      a.buf_len = seq_len - n_flushed;
      if (app) {
        a.k_new = (const uint16_t*)app->k_new; a.v_new = (const uint16_t*)app->v_new;
        a.in_bf16 = app->in_dtype == KVQ_BF16 ? 1 : 0; a.nsb = app->stride_b; a.nsh = app->stride_h;
      }
      a.merge_tag = merge_tag_for(a.rec_splits);
#define KVQ_CASE(BK_, BV_) \
      if (g.bits_k == BK_ && g.bits_v == BV_) return KVQ_CAT(launch_decode_inst_, BK_, BV_)(R, a, plan, stream);
      KVQ_FOR_EACH_PAIR(KVQ_CASE)
#undef KVQ_CASE
      return hipErrorInvalidValue;
    }
    const int32_t records = plan.n_splits + (tail ? 1 : 0);
    // one split of flushed blocks and a tail: the tail's launch, which comes second, takes the first one's record in and
    // writes the result (one launch less than with the merge kernel)
    const bool tail_merges = n_flushed && tail && plan.n_splits == 1;
    a.lens_bound = seq_len; a.lens_block = RL;
    hipError_t e = hipSuccess;
    if (n_flushed) {
      a.seq_len = n_flushed; a.rec_splits = records; a.rec_base = 0; a.lens_mode = 1;
      a.merge_tag = !tail ? merge_tag_for(records) : 0;     // (a launch that writes every record may merge them itself)
#define KVQ_CASE(BK_, BV_) \
      if (g.bits_k == BK_ && g.bits_v == BV_) e = KVQ_CAT(launch_decode_inst_, BK_, BV_)(R, a, plan, stream);
      KVQ_FOR_EACH_PAIR(KVQ_CASE)
#undef KVQ_CASE
      if (e != hipSuccess) return e;
    }
    if (tail) {
      DecodeArgs t = a;
      t.merge_tag = 0;
      t.g.axis_k = KVQ_AXIS_HEAD_DIM; t.g.bits_k = t.g.bits_v = 16; t.g.g_k = t.g.g_v = kHeadDim; t.g.ng_k = t.g.ng_v = 1;
      t.g.rotate_k = 0;                                    // (the buffer holds the input rows: their scores take q itself)
      t.g.resid = 0; t.g.seq_g = 0;
      t.g.t_cap = RL; t.g.page_shift = 0; t.cache.page_table = nullptr;     // (the buffers are per sequence, never paged)
      t.g.kc_stream = t.g.vc_stream = (int64_t)RL * kHeadDim * 2; t.g.km_stream = t.g.vm_stream = 0;
      t.cache.k_codes = c.k_resid; t.cache.v_codes = c.v_resid; t.cache.k_meta = t.cache.v_meta = nullptr;
      if (app) {                                           // (the buffer's newest token comes with this launch)
        t.k_new = (const uint16_t*)app->k_new; t.v_new = (const uint16_t*)app->v_new;
        t.in_bf16 = app->in_dtype == KVQ_BF16 ? 1 : 0; t.nsb = app->stride_b; t.nsh = app->stride_h;
      }
      t.seq_len = tail; t.n_splits = 1; t.steps_per_split = 4; t.lens_mode = 2;
      t.rec_splits = records; t.rec_base = records - 1;
      if (tail_merges) { t.rec_splits = 1; t.rec_base = 0; t.extra_splits = records; }
      e = launch_decode_inst_16_16(R, t, DecodePlan{1, 4, 4}, stream);
      if (e != hipSuccess) return e;
    }
    if (records > 1 && !(n_flushed && !tail) && !tail_merges) {     // (a launch that wrote all the records has merged them itself)
      launch_merge(workspace, out, out_dtype, g.batch * q_heads, records, rot_v_of(g), stream);
      e = hipGetLastError();
    }
    return e;
  }
  a.lens_mode = 0; a.lens_bound = seq_len; a.lens_block = 1;
  a.balance = plan.slots; a.deal_pays = plan.deal_pays;
  if (a.balance) a.rec_splits = deal_records(g, plan.slots);
  a.merge_tag = a.balance ? next_merge_tag()
                          : merge_tag_for(a.rec_splits, !app && a.heads_per_kv > kAloneHeads ? kMergeHereMostAlone : kMergeHereMost);
  if (app) {
    a.k_new = (const uint16_t*)app->k_new; a.v_new = (const uint16_t*)app->v_new;
    a.in_bf16 = app->in_dtype == KVQ_BF16 ? 1 : 0; a.nsb = app->stride_b; a.nsh = app->stride_h;
  }
#define KVQ_CASE(BK_, BV_) \
  if (g.bits_k == BK_ && g.bits_v == BV_) return KVQ_CAT(launch_decode_inst_, BK_, BV_)(R, a, plan, stream);
  KVQ_FOR_EACH_PAIR(KVQ_CASE)
#undef KVQ_CASE
  return hipErrorInvalidValue;
}
#endif

}  // namespace kvq
