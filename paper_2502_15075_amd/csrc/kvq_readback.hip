// Reading the packed planes back row by row (gfx950): dequantize and reconstruction error.
//
// Both kernels are one pass over memory, x^ = code * scale + zero (App. B "Dequantization" of arXiv 2502.15075) in
// between, and should run at the rate of the memory system.  What bounds them is how many loads are in flight: the
// packed bytes of a row are few (112 for K4V2) and sit in four places.  Hence:
//   - keys and values are separate workgroups (blockIdx.z), so that each body is compiled for one tensor's width alone;
//   - the unit is a 32-token block: a thread owns 8 channels of the tokens u and u + 16 of it, whose value codes share
//     their 32-bit words (for widths up to 4), so one set of 8 loads serves two rows;
//   - a workgroup takes several blocks in a row, one or two in registers (codes, scale/zero, reference rows), which are loaded
//     again, no load behind a branch, as soon as a block is done.  (A "next" that is copied to a "current" is waited for in
//     whole at the copy: nothing is in flight from there to the next load, and the copy has registers of its own);
//   - positions come from the grid and a running block number: no division per thread.
// Figures: at the launchers.
#include "kvq_internal.h"
#include "kvq_quantizer.h"

namespace kvq {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Where the two rows (tokens u and u + 16, u < 16) of a value block keep 8 channels d0 .. d0+7 (d0 a multiple of 8): 8 words
// one lane piece apart, from word `dword` of the block; row x4's field starts at bit bit0 + x4 * B * (2 fields apart).
// Widths up to 4: both rows in the same words.  8-bit fields: row 1 in the next word.  16-bit patterns: two words on.
template <int B> constexpr int value_words() { return B <= 4 ? 8 : 16; }
template <int B> __device__ __forceinline__ void load_block_words(const uint8_t* blk, int u, int d0, uint32_t* w) {
  int dw, bit;
  v_field(u, d0, B, &dw, &bit);
  const uint32_t* p = reinterpret_cast<const uint32_t*>(blk) + dw;
  constexpr int LW = B == 1 ? 2 : 4;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    w[e] = p[LW * e];
    if (B == 8) w[8 + e] = p[LW * e + 1];
    if (B == 16) w[8 + e] = p[LW * e + 2];
  }
}
// Row x4's code of channel d0 + e (shift: v_field's bit for token u; the second row's field lies 2 B bits higher)
template <int B> __device__ __forceinline__ uint32_t block_code(const uint32_t* w, int e, int x4, int shift) {
  if (B >= 8) return (w[8 * x4 + e] >> shift) & (B == 16 ? 0xFFFFu : 0xFFu);
  return (w[e] >> (shift + 2 * B * x4)) & ((1u << B) - 1u);
}

// One thread's packed bytes of one 32-token block: 8 channels of two rows.
template <int B, bool IS_V> constexpr int code_words() {
  if (IS_V) return code_hi_bits<B>() ? 2 * 8 : value_words<B>();
  return 2 * (B == 16 ? 4 : B == 8 ? 2 : code_hi_bits<B>() ? 2 : 1);
}
template <int B, bool IS_V, bool KSEQ> struct Packed {
  uint32_t w[code_words<B, IS_V>()];
  uint32_t m[KSEQ ? 8 : 2];           // scale/zero: one entry per row, or (channel-wise keys) one per channel
};

struct Lane { int row, lane16, d0, grp; };         // row 0..15 of the block (and row + 16), channels 8 lane16 .., group

// tv0: the block's first token in plane order (a multiple of 32)
template <int B, bool IS_V, bool KSEQ>
__device__ __forceinline__ void load_packed(Packed<B, IS_V, KSEQ>& p, const Geom& g, const kvq_cache& c, int64_t tv0, const Lane& L) {
  constexpr int LO = code_lo_bits<B>(), HI = code_hi_bits<B>();
  if constexpr (IS_V) {
    const uint8_t* blk = (const uint8_t*)c.v_codes + (tv0 >> 5) * (int64_t)(512 * B);
    load_block_words<LO>(blk, L.row, L.d0, p.w);
    if constexpr (HI != 0) load_block_words<HI>(blk + 512 * LO, L.row, L.d0, p.w + 8);
  } else {
    constexpr int N = code_words<B, IS_V>() / 2;
#pragma unroll
    for (int x4 = 0; x4 < 2; ++x4) {
      const uint8_t* rowp = (const uint8_t*)c.k_codes + (tv0 + L.row + 16 * x4) * (16 * B);
      uint32_t* w = p.w + N * x4;
      if constexpr (B == 16) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(rowp + L.lane16 * 16);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
      } else if constexpr (B == 8) {
        const u32x2 v = *reinterpret_cast<const u32x2*>(rowp + L.lane16 * 8);
        w[0] = v.x; w[1] = v.y;
      } else if constexpr (HI == 0) {
        w[0] = load_bytes<B>(rowp + L.lane16 * B);
      } else {
        const uint8_t* chunk = rowp + (L.lane16 >> 2) * (4 * B);
        w[0] = load_bytes<LO>(chunk + (L.lane16 & 3) * LO);
        w[1] = load_bytes<HI>(chunk + 4 * LO + (L.lane16 & 3) * HI);
      }
    }
  }
  if constexpr (B != 16) {
    const uint32_t* ms = (const uint32_t*)(IS_V ? c.v_meta : c.k_meta);
    if constexpr (KSEQ) {                          // both rows lie in one group: groups are 32 tokens and more
      const u32x4* mp = reinterpret_cast<const u32x4*>(ms + (tv0 / g.seq_g) * kHeadDim + L.d0);
      const u32x4 a = mp[0], b = mp[1];
      p.m[0] = a.x; p.m[1] = a.y; p.m[2] = a.z; p.m[3] = a.w;
      p.m[4] = b.x; p.m[5] = b.y; p.m[6] = b.z; p.m[7] = b.w;
    } else {
      const int ng = IS_V ? g.ng_v : g.ng_k;
      const uint32_t* mp = ms + meta_index(tv0 + L.row, L.grp, ng);
      p.m[0] = mp[0];
      p.m[1] = mp[16 * ng];
    }
  }
}

// Reconstruction of row x4 in binary32 (a 16-bit plane is widened exactly).  code * scale is exact, so the fused
// multiply-add is the one rounding of code * scale + zero.
template <int B, bool IS_V, bool KSEQ>
__device__ __forceinline__ void reconstruct(const Packed<B, IS_V, KSEQ>& p, int x4, int vshift_lo, int vshift_hi, bool raw_bf16,
                                            float val[8]) {
  constexpr int LO = code_lo_bits<B>(), HI = code_hi_bits<B>();
  uint32_t code[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if constexpr (IS_V) {
      code[e] = block_code<LO>(p.w, e, x4, vshift_lo);
      if constexpr (HI != 0) code[e] |= block_code<HI>(p.w + 8, e, x4, vshift_hi) << LO;
    } else {
      constexpr int N = code_words<B, IS_V>() / 2;
      const uint32_t* w = p.w + N * x4;
      if constexpr (B == 16) code[e] = (w[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
      else if constexpr (B == 8) code[e] = (w[e >> 2] >> (8 * (e & 3))) & 0xFFu;
      else if constexpr (HI == 0) code[e] = (w[0] >> (B * e)) & ((1u << B) - 1u);
      else code[e] = ((w[0] >> (LO * e)) & ((1u << LO) - 1u)) | (((w[1] >> (HI * e)) & ((1u << HI) - 1u)) << LO);
    }
  }
  if constexpr (B == 16) {
#pragma unroll
    for (int e = 0; e < 8; ++e) val[e] = widen16((uint16_t)code[e], raw_bf16);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t m = p.m[KSEQ ? e : x4];
      val[e] = __builtin_fmaf((float)code[e], widen16((uint16_t)(m & 0xFFFF), false), widen16((uint16_t)(m >> 16), false));
    }
  }
}

// The wavefront's four rows in the caller's type (one rounding), streaming stores of 1 KB each; the caller's pointer need not
// be aligned beyond its elements.  Row r of the four is token t + r (t: the first; only rows in [t0, t1) are stored), o
// the element offset of row t.  A binary32 row is 32 bytes per lane: it goes through 2 KB of LDS first, so that a store
// covers 1 KB in one piece (two 16-byte stores per lane 32 bytes apart: 27 us, not streaming 18 us, where this takes 13.5: 5 x 8 heads x
// 1835 tokens).
template <int OUT>
__device__ __forceinline__ void store_rows(void* out, int64_t o, int t, int t0, int t1, int lane, const float val[8], float* lds) {
  if constexpr (OUT == KVQ_F32) {
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    typedef float f32x4a4 __attribute__((ext_vector_type(4), aligned(4)));
    f32x4 a = {val[0], val[1], val[2], val[3]}, b = {val[4], val[5], val[6], val[7]};
    f32x4* w = reinterpret_cast<f32x4*>(lds);
    w[2 * lane] = a;
    w[2 * lane + 1] = b;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");     // (LDS is in order within a wavefront; this binds the compiler too)
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const f32x4 v = w[64 * k + lane];
      const int r = 2 * k + (lane >> 5);
      if (t + r >= t0 && t + r < t1)
        __builtin_nontemporal_store((f32x4a4)v, reinterpret_cast<f32x4a4*>((float*)out + o + r * kHeadDim + 4 * (lane & 31)));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  } else {
    const int r = lane >> 4;
    if (t + r < t0 || t + r >= t1) return;
    o += r * kHeadDim + 8 * (lane & 15);
    typedef uint32_t u32x4a2 __attribute__((ext_vector_type(4), aligned(2)));
    u32x4a2 a;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = OUT == KVQ_F16 ? f32_to_f16_bits(val[2 * e]) : f32_to_bf16_bits(val[2 * e]);
      const uint32_t hi = OUT == KVQ_F16 ? f32_to_f16_bits(val[2 * e + 1]) : f32_to_bf16_bits(val[2 * e + 1]);
      a[e] = lo | (hi << 16);
    }
    __builtin_nontemporal_store(a, reinterpret_cast<u32x4a2*>((uint16_t*)out + o));
  }
}

template <int B, bool IS_V, bool KSEQ, int OUT, bool CHAIN>
__device__ __forceinline__ void dequantize_body(const Geom& g, const kvq_cache& c, int32_t t0, int32_t t1, void* out, int32_t chain,
                                                float* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Lane L;
  L.row = threadIdx.x >> 4; L.lane16 = threadIdx.x & 15; L.d0 = 8 * L.lane16;
  L.grp = L.d0 / (IS_V ? g.g_v : g.g_k);
  const int bh = blockIdx.y, b = bh / g.kv_heads, h = bh % g.kv_heads;
  const int first = (t0 >> 5) + blockIdx.x * chain, end = CHAIN ? min(first + chain, ((t1 - 1) >> 5) + 1) : first + 1;
  const bool rotated = IS_V ? g.rotate_v != 0 : g.rotate_k != 0;
  const uint32_t signs = rot_sign_bits(IS_V ? g.signs_v : g.signs_k, L.lane16);
  const bool raw_bf16 = g.raw_dtype == KVQ_BF16;
  int dw, vs_lo = 0, vs_hi = 0;
  if constexpr (IS_V) {
    v_field(L.row, L.d0, code_lo_bits<B>(), &dw, &vs_lo);
    if constexpr (code_hi_bits<B>() != 0) v_field(L.row, L.d0, code_hi_bits<B>(), &dw, &vs_hi);
  }
  if constexpr (!CHAIN) {
    // (a loop of its own, though it has one turn: as the ring below with a depth of one, or with the rows in a function of both, the
    // compiler forms the addresses and orders the rotation otherwise, 2-bit values 1 to 4 % slower, rotated rows up to 10)
    Packed<B, IS_V, KSEQ> cur;
    load_packed(cur, g, c, virtual_token(g, c.page_table, b, h, (int64_t)first * 32), L);
    for (int blk = first; blk < end; ++blk) {
#pragma unroll
      for (int x4 = 0; x4 < 2; ++x4) {
        float val[8];
        reconstruct<B, IS_V, KSEQ>(cur, x4, vs_lo, vs_hi, raw_bf16, val);
        if (rotated) unrotate8(val, L.lane16, signs);            // (uniform; the 16 threads of a row are all here)
        const int t = blk * 32 + 4 * wave + 16 * x4;             // the wavefront's first row
        store_rows<OUT>(out, ((int64_t)bh * (t1 - t0) + (t - t0)) * kHeadDim, t, t0, t1, lane, val, lds + 512 * wave);
      }
    }
  } else {
    constexpr int kDepth = 2;
    Packed<B, IS_V, KSEQ> packed[kDepth];
    auto load_slot = [&](int k, int blk) {                       // (past the end the last block once more)
      load_packed(packed[k], g, c, virtual_token(g, c.page_table, b, h, (int64_t)min(blk, end - 1) * 32), L);
    };
#pragma unroll
    for (int k = 0; k < kDepth; ++k) load_slot(k, first + k);
    for (int blk0 = first; blk0 < end; blk0 += kDepth) {
#pragma unroll
      for (int k = 0; k < kDepth; ++k) {
        const int blk = blk0 + k;
        if (blk < end) {                                         // (uniform)
#pragma unroll
          for (int x4 = 0; x4 < 2; ++x4) {
            float val[8];
            reconstruct<B, IS_V, KSEQ>(packed[k], x4, vs_lo, vs_hi, raw_bf16, val);
            if (rotated) unrotate8(val, L.lane16, signs);
            const int t = blk * 32 + 4 * wave + 16 * x4;
            store_rows<OUT>(out, ((int64_t)bh * (t1 - t0) + (t - t0)) * kHeadDim, t, t0, t1, lane, val, lds + 512 * wave);
          }
        }
        load_slot(k, blk + kDepth);
      }
    }
  }
}

// One body per width, chosen by a uniform branch: KVQ_BODY(width, is it the values', channel-wise keys)
#define KVQ_BY_WIDTH(KVQ_BODY)                                                     \
  if (blockIdx.z == which_v) {                                                     \
    switch (g.bits_v) {                                                            \
      case 1: KVQ_BODY(1, true, false); break;                                     \
      case 2: KVQ_BODY(2, true, false); break;                                     \
      case 3: KVQ_BODY(3, true, false); break;                                     \
      case 4: KVQ_BODY(4, true, false); break;                                     \
      case 6: KVQ_BODY(6, true, false); break;                                     \
      case 8: KVQ_BODY(8, true, false); break;                                     \
      default: KVQ_BODY(16, true, false);                                          \
    }                                                                              \
  } else if (g.axis_k == KVQ_AXIS_SEQ) {                                           \
    switch (g.bits_k) {                                                            \
      case 1: KVQ_BODY(1, false, true); break;                                     \
      case 2: KVQ_BODY(2, false, true); break;                                     \
      case 3: KVQ_BODY(3, false, true); break;                                     \
      case 4: KVQ_BODY(4, false, true); break;                                     \
      case 6: KVQ_BODY(6, false, true); break;                                     \
      default: KVQ_BODY(8, false, true);                                           \
    }                                                                              \
  } else {                                                                         \
    switch (g.bits_k) {                                                            \
      case 1: KVQ_BODY(1, false, false); break;                                    \
      case 2: KVQ_BODY(2, false, false); break;                                    \
      case 3: KVQ_BODY(3, false, false); break;                                    \
      case 4: KVQ_BODY(4, false, false); break;                                    \
      case 6: KVQ_BODY(6, false, false); break;                                    \
      case 8: KVQ_BODY(8, false, false); break;                                    \
      default: KVQ_BODY(16, false, false);                                         \
    }                                                                              \
  }

// which_v: the value of blockIdx.z that stands for the values (1 with both tensors, 0 when only values are asked for)
template <int OUT, bool CHAIN>
__global__ __launch_bounds__(256) void dequantize_kernel(Geom g, kvq_cache c, int32_t t0, int32_t t1, void* k_out, void* v_out,
                                                         int32_t chain, uint32_t which_v) {
  __shared__ __attribute__((aligned(16))) float lds[OUT == KVQ_F32 ? 4 * 512 : 4];
#define KVQ_BODY(B_, V_, S_) dequantize_body<B_, V_, S_, OUT, CHAIN>(g, c, t0, t1, V_ ? v_out : k_out, chain, lds)
  KVQ_BY_WIDTH(KVQ_BODY)
#undef KVQ_BODY
}

// Squared reconstruction error (numerator of the MSE of App. B, "Frobenius Norm (MSE) Perspective") of one tensor: the
// workgroup's blocks, differences and the squares of a thread's 8 channels in binary32, everything above that summed in
// binary64, one atomic add per workgroup (every head's sum is hit by all the workgroups of that head, and atomics on one
// address are served one after the other).
template <int B, bool IS_V, bool KSEQ>
__device__ __forceinline__ void sq_error_body(const Geom& g, const kvq_cache& c, const uint16_t* __restrict__ ref, bool ref_bf16,
                                              int64_t sb, int64_t sh, int64_t st, int32_t t0, int32_t t1,
                                              double* __restrict__ sums, int32_t chain, double* part) {
  Lane L;
  L.row = threadIdx.x >> 4; L.lane16 = threadIdx.x & 15; L.d0 = 8 * L.lane16;
  L.grp = L.d0 / (IS_V ? g.g_v : g.g_k);
  const int bh = blockIdx.y, b = bh / g.kv_heads, h = bh % g.kv_heads;
  const int first = (t0 >> 5) + blockIdx.x * chain, end = min(first + chain, ((t1 - 1) >> 5) + 1);
  const bool rotated = IS_V ? g.rotate_v != 0 : g.rotate_k != 0;
  const uint32_t signs = rot_sign_bits(IS_V ? g.signs_v : g.signs_k, L.lane16);
  const bool raw_bf16 = g.raw_dtype == KVQ_BF16;
  int dw, vs_lo = 0, vs_hi = 0;
  if constexpr (IS_V) {
    v_field(L.row, L.d0, code_lo_bits<B>(), &dw, &vs_lo);
    if constexpr (code_hi_bits<B>() != 0) v_field(L.row, L.d0, code_hi_bits<B>(), &dw, &vs_hi);
  }
  const int64_t base = (int64_t)b * sb + (int64_t)h * sh + L.d0;
  // the reference rows of tokens row, row + 16 of block blk (rows outside [t0, t1) re-read the nearest row inside)
  auto load_ref = [&](u32x4 (&r)[2], int blk) {
#pragma unroll
    for (int x4 = 0; x4 < 2; ++x4) {
      const int t = min(max(blk * 32 + L.row + 16 * x4, t0), t1 - 1);
      r[x4] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ref + base + (int64_t)(t - t0) * st));
    }
  };
  u32x4 rows[2];
  Packed<B, IS_V, KSEQ> packed;
  load_ref(rows, first);
  load_packed(packed, g, c, virtual_token(g, c.page_table, b, h, (int64_t)first * 32), L);
  double acc = 0.0;
  for (int blk = first; blk < end; ++blk) {
#pragma unroll
    for (int x4 = 0; x4 < 2; ++x4) {
      float val[8], x[8];
      reconstruct<B, IS_V, KSEQ>(packed, x4, vs_lo, vs_hi, raw_bf16, val);
      const uint32_t rw[4] = {rows[x4].x, rows[x4].y, rows[x4].z, rows[x4].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), ref_bf16);
      // rotated rows are compared in the rotated basis: ||R x - y||_2 = ||x - R^T y||_2
      if (rotated) rotate8(x, L.lane16, signs);
      float sq = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float err = x[e] - val[e];
        sq += err * err;
      }
      const int t = blk * 32 + L.row + 16 * x4;
      if (t >= t0 && t < t1) acc += (double)sq;                // (what lies outside may hold anything)
    }
    // the next block into the same registers, the loads moved up by the compiler to where each is used for the last time (past
    // the end the last block once more, so that none is behind a branch)
    const int nb = min(blk + 1, end - 1);
    load_ref(rows, nb);
    load_packed(packed, g, c, virtual_token(g, c.page_table, b, h, (int64_t)nb * 32), L);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    const double v = (part[0] + part[1]) + (part[2] + part[3]);
    if (v != 0.0) atomicAdd(sums + (int64_t)bh * 2 + (IS_V ? 1 : 0), v);
  }
}

// (one kernel per pair of widths: with a uniform switch over the widths inside, as the dequantize kernel has it, the widest
// body's registers cost the narrow ones a third of their wavefronts)
template <int BK, int BV, bool KSEQ>
__global__ __launch_bounds__(256) void sq_error_kernel(Geom g, kvq_cache c, const uint16_t* __restrict__ k_ref,
                                                       const uint16_t* __restrict__ v_ref, int ref_bf16, int64_t sb,
                                                       int64_t sh, int64_t st, int32_t t0, int32_t t1,
                                                       double* __restrict__ sums, int32_t chain, uint32_t which_v) {
  __shared__ double part[4];
  if (blockIdx.z == which_v) sq_error_body<BV, true, false>(g, c, v_ref, ref_bf16 != 0, sb, sh, st, t0, t1, sums, chain, part);
  else sq_error_body<BK, false, KSEQ>(g, c, k_ref, ref_bf16 != 0, sb, sh, st, t0, t1, sums, chain, part);
}

__global__ __launch_bounds__(256) void zero_f64_kernel(double* p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

}  // namespace

// Dequantize, bound by its stores.  Blocks per workgroup: one for binary32 rows and for calls of fewer than 24576 blocks (both tensors
// counted), which need their workgroups side by side; above that eight in a row, four of some keys alone (deq_in_a_row), dealt out evenly,
// two of them in registers.  From 16384 blocks on already where one round of workgroups less pays: narrow tensors, and middling ones in
// long sequences, whose uneven last share is a small part.
// In turn, to bf16, us with one / four / eight in a row (and with the version before: four, the next copied to the current, from 24576 on).
// Both tensors:
//   8 x 8 heads x 8192 tokens (32768 blocks)  K4V2 60.4 / 53.5 / 50.7 (54.0)  K8V8 67.4 / 71.0 / 68.4 (72.7)  unquantized 156.0 / 179.2 / 164.0 (179.9)
//   8 x 8 x 32768 (131072)                    K4V2 228.6 / 204.8 / 191.0 (204.7)
//   8 x 8 x 5000 (20096)                      K4V2 37.1 / 33.3 / 32.5  paged 39.1 / 37.5 / 36.4  K4V4 42.2 / 41.4 / 41.0  K8V8 42.2 / 44.9 / 43.5
//                                             unquantized 96.9 / 112.3 / 103.1
//   40 x 8 x 900 (18560)                      K4V2 33.6 / 32.6 / 33.1  paged 35.8 / 37.2 / 38.3  rotated keys 40.1 / 41.8 / 42.5
//                                             K4V4 38.4 / 40.4 / 39.1  K8V8 39.1 / 45.3 / 43.3  unquantized 89.9 / 112.5 / 103.5
// Keys alone:
//   16384 blocks   K4 29.8 / 25.7 / 27.7  K8 30.8 / 32.2 / 32.9
//   32768          K4 57.8 / 49.2 / 51.3 (50.4)  K2 57.3 / 47.4 / 45.4 (49.5)  unquantized 80.7 / 78.3 / 80.5 (79.0)
//   65536          K4 115.9 / 97.8 / 96.4 (97.9)  K2 113.8 / 94.8 / 91.6 (97.9)  unquantized 177.1 / 180.1 / 195.4 (187.1)
// Values alone:
//   16384          V2 29.2 / 28.2 / 27.3  V8 39.6 / 42.7 / 39.8
//   32768          V2 59.3 / 53.8 / 51.4 (55.8)
// To binary32, whose workgroups write twice the bytes: 8 x 8 x 8192 85.5 us with one, 99.4 with eight, 101 with four; x 5000 56.4 and 63.6;
// 20 x 8 x 3000 87.3, 93 with four.  Streaming stores: 16-bit rows 52 us with them, 87 without.
constexpr int kDeqChain = 8, kDeqChainKeys = 4, kDeqChainFrom = 24576, kDeqChainFromNarrow = 16384, kDeqLong = 64, kDeqManyKeys = 49152;
// Whether several in a row pay from the smaller number of blocks on (blocks: of one sequence).
inline bool deq_chains_early(const Geom& g, bool keys, bool values, int blocks) {
  if (!values) return g.bits_k <= 6 && !g.rotate_k;
  if (!keys) return g.bits_v <= 2;
  if (g.bits_k <= 4 && g.bits_v <= 2 && !g.rotate_k && !g.rotate_v && g.page_shift == 0) return true;
  return blocks >= kDeqLong && (g.bits_v <= 4 || (g.bits_v == 8 && g.bits_k <= 4));
}
// How many at most (blocks: of the call).
inline int deq_in_a_row(const Geom& g, bool values, int64_t blocks) {
  if (values) return kDeqChain;
  if (g.bits_k >= 8 || g.rotate_k) return kDeqChainKeys;
  return g.bits_k >= 4 && g.axis_k != KVQ_AXIS_SEQ && g.page_shift == 0 && blocks < kDeqManyKeys ? kDeqChainKeys : kDeqChain;
}
hipError_t launch_dequantize(const Geom& g, const kvq_cache& c, int32_t t0, int32_t t1, void* k_out, void* v_out,
                             int out_dtype, hipStream_t stream) {
  if (t1 == t0) return hipSuccess;
  const int streams = g.batch * g.kv_heads, blocks = ((t1 - 1) >> 5) - (t0 >> 5) + 1;
  const int tensors = (k_out ? 1 : 0) + (v_out ? 1 : 0);
  const uint32_t which_v = k_out ? 1u : 0u;
  const int64_t all = (int64_t)blocks * streams * tensors;
  const bool early = deq_chains_early(g, k_out != nullptr, v_out != nullptr, blocks);
  const bool chained = out_dtype != KVQ_F32 && all >= (early ? kDeqChainFromNarrow : kDeqChainFrom);
  const int most = deq_in_a_row(g, v_out != nullptr, all);
  const int per = chained ? (blocks + most - 1) / most : blocks, chain = (blocks + per - 1) / per;
  const dim3 grid((blocks + chain - 1) / chain, streams, tensors);
#define KVQ_DEQ_LAUNCH(OUT_)                                                                                              \
  if (OUT_ != KVQ_F32 && chained)                                                                                        \
    hipLaunchKernelGGL((dequantize_kernel<OUT_, OUT_ != KVQ_F32>), grid, dim3(256), 0, stream, g, c, t0, t1, k_out, v_out, chain, which_v); \
  else                                                                                                                   \
    hipLaunchKernelGGL((dequantize_kernel<OUT_, false>), grid, dim3(256), 0, stream, g, c, t0, t1, k_out, v_out, chain, which_v)
  if (out_dtype == KVQ_F32) { KVQ_DEQ_LAUNCH(KVQ_F32); }
  else if (out_dtype == KVQ_F16) { KVQ_DEQ_LAUNCH(KVQ_F16); }
  else { KVQ_DEQ_LAUNCH(KVQ_BF16); }
#undef KVQ_DEQ_LAUNCH
  return hipGetLastError();
}

// Reconstruction error.  One round of workgroups, 4 per compute unit, each walking its share of a stream's blocks; at most
// 32 workgroups per stream and tensor, because they all add to one address (209 of them: 32 us for 6685 tokens of 8
// heads, 32 of them: 12 us), or one per 16 blocks where that is more, so that a long stream is not walked by few of them
// (K4V2, one head, 65536 tokens: 60 us with 32, 33, 19 and 16 us with one per 32, 16 and 8 blocks; 4 heads keys alone 48,
// 29, 23 and 27; 8 heads x 131072 122, and 115 with all three; the first version 56, 105 and 166).  Measured, K4V2, 8 x 8 heads x 32768 tokens, with the copied block: 226 us = 5.8 TB/s (3, 5, 6, 7 per unit: 233, 239,
// 228, 237; 8 and 16 per unit, more than are resident at once: 251 and 243); 13 x 8 x 2378, K4V1: 36 us (5 to 7 per unit:
// 33, 33, 35).  Before (one row at a time per thread, 8192 workgroups): 291 us, 40 us for the 6685 tokens, 50 us.
// One block in registers, loaded again in place, in turn with a next block that is copied to the current one: 8 x 8 heads x 32768 tokens 216 and 203 us
// (228 and 216 on another card: 5.8 and 6.1 TB/s); 8 x 8 x 8192 K3V2 64.5 and 60.2, K8V4 64.2 and 62.2, K4V6 81 and 74, rotated keys 78 and 74; 48 x
// 8 x 2000, K8V8, 111 and 95; one head of 65536 tokens 18.6 and 16.7; 33 x 8 x 4096 135 and 131; 44 x 8 x 4096 160 and 154.  Two blocks so: 8 x 8 x
// 32768 205, but 94 registers instead of 67 leave five workgroups per unit where six or seven were resident: 44 x 8 x 4096 163, 43 x 8 x 2000, K8V4, 99
// (93 copied, 90.5 with one).  Loaded at the head of the loop instead: 3 x 8 x 30000, K2V2, 95 (80 and 75), one head of 65536 21.3.
// The share is rounded down, which leaves up to a third of the round empty, except where it would be one workgroup per
// stream and tensor and leave a quarter or more empty: two are taken there, up to 6 per unit, all resident at once.  528
// streams and tensors of 4096 tokens 135 us with two, 166 with one (152 before); 704: 166 and 170; 832: 219 and 212.
// Rounded to the nearest, 176 to 448 streams and tensors lose up to 9 % (384: 20.4 against 18.7 us).
constexpr int kErrPerUnit = 4, kErrPerStream = 32, kErrBlocks = 16;
constexpr int error_workgroups(int64_t pairs, int64_t round, int64_t blocks) {     // pairs of stream and tensor; workgroups of one round
  int64_t per = round / pairs;
  if (per <= 1) per = 4 * pairs <= 3 * round ? 2 : 1;
  const int64_t most = blocks / kErrBlocks > kErrPerStream ? blocks / kErrBlocks : kErrPerStream;
  return (int)(per < most ? per : most);
}
constexpr bool error_rounds_are_full(int64_t round) {
  for (int64_t pairs = round / kErrPerStream; pairs <= round; ++pairs) {
    const int64_t n = error_workgroups(pairs, round, 0) * pairs;
    if (3 * n < 2 * round || 2 * n > 3 * round) return false;
  }
  return true;
}
static_assert(error_rounds_are_full(1024) && error_rounds_are_full(4 * 304) && error_rounds_are_full(4 * 32), "two thirds of a round to one and a half");
static_assert(error_workgroups(2, 1024, 2048) == 128 && error_workgroups(2, 1024, 209) == 32, "long streams take more than 32");

hipError_t launch_reconstruction_error(const Geom& g, const kvq_cache& c, const void* k_ref, const void* v_ref,
                                       int ref_dtype, int64_t sb, int64_t sh, int64_t st, int32_t t0, int32_t t1,
                                       double* sums, hipStream_t stream) {
  const int streams = g.batch * g.kv_heads;
  const int64_t n = (int64_t)streams * 2;
  // cleared by a kernel, not a memset, so that the call can be captured into a graph
  hipLaunchKernelGGL(zero_f64_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, sums, n);
  if (t1 == t0) return hipGetLastError();
  const int blocks = ((t1 - 1) >> 5) - (t0 >> 5) + 1;
  const int tensors = (k_ref ? 1 : 0) + (v_ref ? 1 : 0);
  const int per = error_workgroups((int64_t)streams * tensors, (int64_t)kErrPerUnit * device_compute_units(), blocks);
  const int chain = (blocks + per - 1) / per;
  const dim3 grid((blocks + chain - 1) / chain, streams, tensors);
#define KVQ_ERR_LAUNCH(BK_, BV_, S_)                                                                                     \
  hipLaunchKernelGGL((sq_error_kernel<BK_, BV_, S_>), grid, dim3(256), 0, stream, g, c, (const uint16_t*)k_ref,          \
                     (const uint16_t*)v_ref, ref_dtype == KVQ_BF16 ? 1 : 0, sb, sh, st, t0, t1, sums, chain, k_ref ? 1u : 0u)
#define KVQ_ERR_CASE(BK_, BV_)                                                                                          \
  if (g.bits_k == BK_ && g.bits_v == BV_) {                                                                             \
    if constexpr (BK_ != 16 && BV_ != 16) {        /* (channel-wise keys: both tensors quantized) */                    \
      if (g.axis_k == KVQ_AXIS_SEQ) KVQ_ERR_LAUNCH(BK_, BV_, true);                                                     \
      else KVQ_ERR_LAUNCH(BK_, BV_, false);                                                                             \
    } else {                                                                                                            \
      KVQ_ERR_LAUNCH(BK_, BV_, false);                                                                                  \
    }                                                                                                                   \
  }
#define KVQ_ERR_ROW(BK_) KVQ_ERR_CASE(BK_, 1) KVQ_ERR_CASE(BK_, 2) KVQ_ERR_CASE(BK_, 3) KVQ_ERR_CASE(BK_, 4) \
  KVQ_ERR_CASE(BK_, 6) KVQ_ERR_CASE(BK_, 8) KVQ_ERR_CASE(BK_, 16)
  KVQ_ERR_ROW(1) KVQ_ERR_ROW(2) KVQ_ERR_ROW(3) KVQ_ERR_ROW(4) KVQ_ERR_ROW(6) KVQ_ERR_ROW(8) KVQ_ERR_ROW(16)
#undef KVQ_ERR_ROW
#undef KVQ_ERR_CASE
#undef KVQ_ERR_LAUNCH
  return hipGetLastError();
}

}  // namespace kvq
