// Staging of value codes on their way into the planes, shared by the append kernels: streaming accesses, the LDS area that
// holds one element per code in storage order, and the assembly of output words from it.
#pragma once
#include "kvq_internal.h"
#include "kvq_quantizer.h"

namespace kvq {
namespace {

constexpr int kSpan = 64;                // tokens one workgroup covers (two 32-token value blocks)

// LDS staging of the value codes of one span, already in storage order: one element per code, the F = 32/b_V codes
// of an output word adjacent (so a word is assembled from one wide LDS read).  (Padding the area against the bank
// conflicts of the strided byte writes was measured: its address arithmetic costs more than the conflicts, 3 %.)

// 16 bytes read once / written once: streaming accesses (see store_bytes)
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
  const u32x4v v = __builtin_nontemporal_load(reinterpret_cast<const u32x4v*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream16(void* p, uint4 w) {
  typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
  u32x4v v; v.x = w.x; v.y = w.y; v.z = w.z; v.w = w.w;
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4v*>(p));
}

// Pack the codes held one per byte in w (first code in the lowest byte) into adjacent b-bit fields.
// (Bytes of tokens that were not staged hold garbage: they are masked to b bits so that they stay inside their field.)
template <int B> __device__ __forceinline__ uint32_t pack_bytes(uint32_t w) {
  if (B == 1) { w &= 0x01010101u; return (w | (w >> 7) | (w >> 14) | (w >> 21)) & 0xFu; }
  if (B == 2) { w &= 0x03030303u; return (w | (w >> 6) | (w >> 12) | (w >> 18)) & 0xFFu; }
  if (B == 4) return (w & 0xFu) | ((w >> 4) & 0xF0u) | ((w >> 8) & 0xF00u) | ((w >> 12) & 0xF000u);
  return w;
}

// Token row (0..63 of the span) -> (block, word family, field): the codes of the 8 channels d0..d0+7 of this lane go
// to 8 words one lane piece (LW = 4 words, 2 for 1-bit codes) apart; they are staged in LDS in storage order, one
// element per code.
template <int BV>
__device__ __forceinline__ void stage_value_codes(uint8_t* vstage, int row, int d0, const uint32_t codes[8]) {
  constexpr int F = 32 / BV, P = 16 / BV, ES = BV == 16 ? 2 : 1, LW = BV == 1 ? 2 : 4;
  const int sub = row >> 5, u = row & 31;
  const int j = (u >> 2) & 3, i = 4 * (u >> 4) + (u & 3);
  const int x = i & 1, v = i >> 1;
  const int q = 4 * (d0 >> 4) + v;
  const int e_idx = q / P, p = q % P;
  const int word0 = sub * (128 * BV) + (BV == 1 ? 0 : (e_idx >> 2) * 256) + (16 * j + (d0 & 15)) * LW + (e_idx & (LW - 1));
  const int a0 = (word0 * F + x * P + p) * ES;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int a = a0 + e * LW * F * ES;
    if (BV == 16) *reinterpret_cast<uint16_t*>(vstage + a) = (uint16_t)codes[e];
    else vstage[a] = (uint8_t)codes[e];
  }
}

// Assemble a 32-bit word of the span from its staged codes.
template <int BV> __device__ __forceinline__ uint32_t staged_word(const uint8_t* sp) {
  if (BV == 1) {
    const uint4 r0 = *reinterpret_cast<const uint4*>(sp), r1 = *reinterpret_cast<const uint4*>(sp + 16);
    return pack_bytes<1>(r0.x) | (pack_bytes<1>(r0.y) << 4) | (pack_bytes<1>(r0.z) << 8) | (pack_bytes<1>(r0.w) << 12) |
           (pack_bytes<1>(r1.x) << 16) | (pack_bytes<1>(r1.y) << 20) | (pack_bytes<1>(r1.z) << 24) | (pack_bytes<1>(r1.w) << 28);
  } else if (BV == 2) {
    const uint4 r = *reinterpret_cast<const uint4*>(sp);
    return pack_bytes<2>(r.x) | (pack_bytes<2>(r.y) << 8) | (pack_bytes<2>(r.z) << 16) | (pack_bytes<2>(r.w) << 24);
  } else if (BV == 4) {
    const uint2 r = *reinterpret_cast<const uint2*>(sp);
    return pack_bytes<4>(r.x) | (pack_bytes<4>(r.y) << 16);
  }
  return *reinterpret_cast<const uint32_t*>(sp);              // 8-bit: four codes; 16-bit: two patterns
}
// One thread per 32-bit word of the span (two blocks of 128*BV words, BW words apart in the plane: a block of 3- or
// 6-bit codes is a block of low parts followed by a block of high parts): assemble the word from the staged codes and
// store it; when the span is only partly covered by the new tokens [lo, hi), keep the fields of the other tokens.
template <int BV, int BW = 128 * BV, int SPAN = kSpan, bool NT = false>
__device__ __forceinline__ void store_value_words(uint32_t* vcp, const uint8_t* vstage, int tid, int lo, int hi) {
  constexpr int F = 32 / BV, P = 16 / BV, ES = BV == 16 ? 2 : 1, W = 128 * BV, N = SPAN / 32 * W;
  static_assert(BV != 16 || (BW == W && N % 256 == 0), "16-bit patterns: blocks follow each other, whole rounds of words");
  if (lo == 0 && hi == SPAN) {                                 // (uniform; a path of its own, or the masks below are formed here too)
#pragma unroll
    for (int w0 = 0; w0 < N; w0 += 256) {
      const int w = w0 + tid;
      if (N % 256 != 0 && w >= N) break;
      uint32_t* vc = vcp + (w / W) * (BW - W) + w;             // the word's place in the plane
      const uint32_t bits = staged_word<BV>(vstage + w * F * ES);
      if (NT) __builtin_nontemporal_store(bits, vc); else *vc = bits;
    }
    return;
  }
  // partially covered span: keep the fields of tokens outside [lo, hi)
  auto fields = [&](int w) -> uint32_t {                       // those of word w that belong to tokens inside
    const int sub = w / W, wi = w % W;
    const int piece = wi >> 8, rem = wi & 255;
    const int L = BV == 1 ? wi >> 1 : rem >> 2, m = BV == 1 ? wi & 1 : rem & 3;
    const int e_idx = 4 * piece + m;
    const int j = L >> 4;
    const uint32_t fmask = BV == 16 ? 0xFFFFu : ((1u << BV) - 1u);
    uint32_t mask = 0;
    for (int x = 0; x < 2; ++x)
      for (int p = 0; p < P; ++p) {
        const int q = e_idx * P + p;
        const int v = q & 3;
        const int i = 2 * v + x;
        const int tt = 32 * sub + 16 * (i >> 2) + 4 * j + (i & 3);
        if (tt >= lo && tt < hi) mask |= fmask << (16 * x + BV * p);
      }
    return mask;
  };
  if constexpr (BV == 16) {
    // 8 words per thread: their present contents are loaded up front, whether needed or not.  Behind the test of the mask the
    // loads come one after the other: 32 x 8 heads x 500 tokens from position 5, K4V16, 29.3 us that way and 24.1 this way
    // (27.4 before full spans had a path of their own).  With fewer words per thread it does not pay (8-bit codes: the full
    // spans of the same kernel lose 2 % to the registers).
    uint32_t old[N / 256];
#pragma unroll
    for (int k = 0; k < N / 256; ++k) old[k] = vcp[256 * k + tid];       // (BW == W)
#pragma unroll
    for (int k = 0; k < N / 256; ++k) {
      const int w = 256 * k + tid;
      const uint32_t mask = fields(w);
      if (mask != 0) vcp[w] = (staged_word<BV>(vstage + w * F * ES) & mask) | (old[k] & ~mask);
    }
  } else {
    for (int w = tid; w < N; w += 256) {
      uint32_t* vc = vcp + (w / W) * (BW - W);
      const uint32_t bits = staged_word<BV>(vstage + w * F * ES);
      const uint32_t mask = fields(w);
      if (mask == 0) continue;
      vc[w] = (bits & mask) | (vc[w] & ~mask);
    }
  }
}

// Bytes of LDS that stage the codes of one span: one staging area per part of a code (3- and 6-bit value codes are a
// low part and a high part, each packed into a block of its own).
template <int BV, int SPAN = kSpan> constexpr int stage_area() { return SPAN * kHeadDim * (BV == 16 ? 2 : 1); }
template <int BV, int SPAN = kSpan> constexpr int stage_total() { return stage_area<BV, SPAN>() * (code_hi_bits<BV>() ? 2 : 1); }

template <int BV, int SPAN = kSpan>
__device__ __forceinline__ void stage_value_row(uint8_t* vstage, int row, int d0, const uint32_t codes[8]) {
  constexpr int VLO = code_lo_bits<BV>(), VHI = code_hi_bits<BV>();
  if constexpr (VHI == 0) {
    stage_value_codes<BV>(vstage, row, d0, codes);
  } else {                                         // (the low parts are cut to their field when the words are packed)
    uint32_t high[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) high[e] = codes[e] >> VLO;
    stage_value_codes<VLO>(vstage, row, d0, codes);
    stage_value_codes<VHI>(vstage + stage_area<BV, SPAN>(), row, d0, high);
  }
}

// vc: the span's first block in the plane
template <int BV, int SPAN = kSpan, bool NT = false>
__device__ __forceinline__ void store_value_span(uint32_t* vc, const uint8_t* vstage, int tid, int lo, int hi) {
  constexpr int VLO = code_lo_bits<BV>(), VHI = code_hi_bits<BV>();
  if constexpr (VHI == 0) {
    store_value_words<BV, 128 * BV, SPAN, NT>(vc, vstage, tid, lo, hi);
  } else {
    store_value_words<VLO, 128 * BV, SPAN, NT>(vc, vstage, tid, lo, hi);
    store_value_words<VHI, 128 * BV, SPAN, NT>(vc + 128 * VLO, vstage + stage_area<BV, SPAN>(), tid, lo, hi);
  }
}

}  // namespace
}  // namespace kvq
