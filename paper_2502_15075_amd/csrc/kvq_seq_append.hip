// Append kernel of caches with a residual buffer: channel-wise key groups, or token-wise keys behind a buffer (gfx950).
//
// The quantizer's arithmetic is that of the token-wise append (App. B of arXiv 2502.15075, exact statement in kvq.h); this
// file too is compiled with floating-point contraction off.
#include "kvq_stage.h"

// Compiled twice: with KVQ_SA_QUADS the kernels that store value patterns four tokens at a time, without it those that store
// them one by one, and the launchers.
#ifdef KVQ_SA_QUADS
#define KVQ_QUADS true
#else
#define KVQ_QUADS false
#endif

namespace kvq {
namespace {

// The 16-bit patterns of channels d0 .. d0+7 (d0 a multiple of 8) of value row t of a residual buffer.
__device__ __forceinline__ void value_patterns8(const uint8_t* vr, int t, int d0, uint32_t code[8]) {
  int dw, bit;
  v_field(t & 31, d0, 16, &dw, &bit);
  const uint32_t* blk = reinterpret_cast<const uint32_t*>(vr + (t >> 5) * (512 * 16)) + dw;
#pragma unroll
  for (int e = 0; e < 8; ++e) code[e] = (blk[4 * e] >> bit) & 0xFFFFu;
}

// Minimum and maximum of x over the four 16-lane rows of a wavefront, in every lane: each swap of rows (of halves) leaves the
// two values to compare in the two registers.
__device__ __forceinline__ float rows_min(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = min2f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return min2f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float rows_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float m = max2f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return max2f(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Value patterns of four neighbouring tokens into the residual buffer's block of 32 (v_field's order for 16-bit patterns: a channel's
// 8 tokens 4 j .. 4 j + 3 of both 16-token tiles are 16 bytes).  A wavefront's four rows of lanes hold the four tokens, 8 channels
// a lane; a transposition of 4 x 4 words by two swaps of rows and two of halves leaves every lane with two channels of all four,
// which go out as 16 bytes each, or 8 where only one tile's tokens are there.  As 16-bit stores 16 bytes apart they were one
// request of the second-level cache each, 8192 a block and sequence: 43 x 8 heads x 2036 tokens, where the last blocks of all
// sequences fall to one of the 8 parts of the chip, 174 us and 90 so, 35 x 8 x 776 36.5 and 31.4, 11 x 8 x 1921 25.3 and 23.6.  Every lane takes part.
//   a, b  this lane's rows of the two tiles; put_a, put_b: whether all four tokens of the tile are stored (uniform)
__device__ __forceinline__ void store_value_quads(uint8_t* block, int j, int lane16, int r, const uint4& a, const uint4& b, bool put_a, bool put_b) {
  auto pairs = [](const uint4& x, uint2 (&ch)[2]) {
    const auto s0 = __builtin_amdgcn_permlane16_swap(x.x, x.y, false, false), s1 = __builtin_amdgcn_permlane16_swap(x.z, x.w, false, false);
    const auto e = __builtin_amdgcn_permlane32_swap(s0[0], s1[0], false, false), o = __builtin_amdgcn_permlane32_swap(s0[1], s1[1], false, false);
    // e[0], o[0], e[1], o[1]: word r of tokens 0 .. 3
    ch[0] = make_uint2((e[0] & 0xFFFFu) | (o[0] << 16), (e[1] & 0xFFFFu) | (o[1] << 16));
    ch[1] = make_uint2((e[0] >> 16) | (o[0] & 0xFFFF0000u), (e[1] >> 16) | (o[1] & 0xFFFF0000u));
  };
  uint2 ca[2], cb[2];
  pairs(a, ca);
  pairs(b, cb);
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int c = 8 * lane16 + 2 * r + k;
    uint32_t* dst = reinterpret_cast<uint32_t*>(block) + (c >> 4) * 256 + (16 * j + (c & 15)) * 4;
    if (put_a && put_b) *reinterpret_cast<uint4*>(dst) = make_uint4(ca[k].x, ca[k].y, cb[k].x, cb[k].y);
    else if (put_a) *reinterpret_cast<uint2*>(dst) = ca[k];
    else *reinterpret_cast<uint2*>(dst + 2) = cb[k];
  }
}

// Channel-wise keys (Sec. 4 "Downstream Task Accuracy": the per-column back-end with its residual buffer).
// One workgroup = one block of RLT tokens (the residual buffer's length: 64 or 128) of one (b,h) stream, restricted to
// the new tokens [lo, hi) in it.  New tokens that no later token of this call overwrites go to their residual slot as
// 16-bit patterns.  A block that this call completes is flushed: rows below lo come back from the residual buffer (the
// launcher makes sure that no other workgroup of the same launch writes there), keys are quantized channel by channel
// (a group is g.seq_g = 32, 64 or 128 consecutive tokens of one channel, RLT / g.seq_g groups per channel and block),
// values token-wise exactly as in quantize_append_kernel.
// QUADS: value patterns go to the buffer four tokens at a time where four stay (store_value_quads), the others one by one.
// KTOK: the keys of a flushed block are quantized row by row like the values (a residual buffer in front of token-wise
// keys); otherwise channel by channel.
// What bounds it: vector instructions (with rotated keys about 1300 per thread and 64-token block) and memory in about equal
// parts.  Hence stores stream (loads: see launch_sa), rows are compared and rotated by register permutes, and a channel's scale, zero and
// reciprocal are formed once per workgroup instead of by every thread that holds the channel.  8 x 8 heads x 8229 tokens,
// K4V2: with rotated keys 111 us before and 78 us now (4.2 TB/s), without 81 and 64 us.  (Several blocks per workgroup with
// the next one's rows loaded ahead, which pays in quantize_append_kernel, costs this one its occupancy: 210 registers,
// 115 us with rotated keys at 2 wavefronts per unit's SIMD, 126 at 3.)
template <int BK, int BV, bool BF, bool KTOK, int RLT, bool STREAM_IN, bool QUADS>
__global__ __launch_bounds__(256) void seq_append_kernel(Geom g, kvq_cache c, const uint16_t* __restrict__ k_new,
                                                         const uint16_t* __restrict__ v_new, int64_t sb, int64_t sh,
                                                         int64_t st, int32_t pos, int32_t n_new,
                                                         const int32_t* __restrict__ pos_arr, int32_t max_pos) {
  static_assert(RLT % kSpan == 0, "a flushed block is a whole number of value spans");
  constexpr int NIT = RLT / 16;                            // rows per thread: rg, rg + 16, ...
  constexpr int NGR = RLT / 32;                            // the most key groups a block can hold
  __shared__ __attribute__((aligned(16))) uint8_t vstage[stage_total<BV>()];
  __shared__ __attribute__((aligned(16))) float s_mn[KTOK ? 1 : NGR][4][kHeadDim], s_mx[KTOK ? 1 : NGR][4][kHeadDim];
  __shared__ __attribute__((aligned(16))) float s_zero[KTOK ? 1 : NGR][kHeadDim], s_rcp[KTOK ? 1 : NGR][kHeadDim];
  const int tid = threadIdx.x;
  const int bh = blockIdx.y;
  const int b = bh / g.kv_heads, h = bh % g.kv_heads;
  if (pos_arr) pos = min(max(pos_arr[b], 0), max_pos);     // one token per sequence at its own position (n_new == 1)
  // Where the blocks of a sequence are a multiple of 8, its last two, which fill the buffer, would fall to the same part of the chip for all
  // sequences: they begin at another one each there (43 x 8 heads x 2036 tokens 89.7 us without, 83.0; 128-token buffers, 10 x 8 x 1937, 31.9
  // and 26.5).  With 8, 16, 32, 64, 128, 256 and 512 blocks, without and with it, 8 kv heads: 32 x 500 tokens 25.2 and 24.0, 32 x 1012 42.0 and 38.0, 32 x
  // 2036 72.3 and 66.9, 32 x 4084 125.6 and 124.4, 16 x 8180 121.4 and 119.8, 8 x 16372 121.7 and 120.4, 1 x 32756 36.9 and 36.6; of few sequences between
  // 1 % more and 7 % less.  Elsewhere the parts share them anyway, and the order costs (8 x 8 x 8229 61.9 and 64.3).
  int turn = blockIdx.x;
  if constexpr (QUADS) {
    if ((gridDim.x & 7) == 0) {                            // (uniform)
      turn += blockIdx.y & 7;
      if (turn >= (int)gridDim.x) turn -= gridDim.x;
    }
  }
  const int blk = pos / RLT + turn;
  const int lo = max(pos, blk * RLT) - blk * RLT;
  const int hi = min(pos + n_new, (blk + 1) * RLT) - blk * RLT;
  const bool complete = hi == RLT;                         // this call brings the block's last token
  const int lane16 = tid & 15, rg = tid >> 4;
  const int d0 = lane16 * 8;
  uint8_t* kr = (uint8_t*)c.k_resid + (int64_t)bh * (RLT * kHeadDim * 2);
  uint8_t* vr = (uint8_t*)c.v_resid + (int64_t)bh * (RLT * kHeadDim * 2);

  // the rows rg + 16 it; no load is conditional (rows outside the new tokens re-read the nearest one inside)
  uint4 kraw[NIT], vraw[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int row = min(max(rg + 16 * it, lo), hi - 1);
    const int64_t src = (int64_t)b * sb + (int64_t)h * sh + ((int64_t)blk * RLT + row - pos) * st + d0;
    if constexpr (STREAM_IN) {
      kraw[it] = load_stream16(k_new + src);
      vraw[it] = load_stream16(v_new + src);
    } else {
      kraw[it] = *reinterpret_cast<const uint4*>(k_new + src);
      vraw[it] = *reinterpret_cast<const uint4*>(v_new + src);
    }
  }
  // the rows [keep, hi) are the last tokens of this call that land in their slots
  const int keep = max(lo, pos + n_new - RLT - blk * RLT);
  const int quad = 4 * __builtin_amdgcn_readfirstlane(tid >> 6);           // a wavefront's rows: 16 it + quad .. + 3
  if constexpr (QUADS) {
    if (keep < hi) {                                       // (uniform)
#pragma unroll
      for (int it = 0; it < NIT; it += 2) {
        const bool full0 = 16 * it + quad >= keep && 16 * it + quad + 4 <= hi, full1 = 16 * it + quad + 16 >= keep && 16 * it + quad + 20 <= hi;
        if (full0 || full1) store_value_quads(vr + (it >> 1) * (512 * 16), quad >> 2, lane16, rg & 3, vraw[it], vraw[it + 1], full0, full1);
      }
    }
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int row = rg + 16 * it;
    if (row >= lo && row < hi) {
      if (row >= keep) {
        *reinterpret_cast<uint4*>(kr + row * (kHeadDim * 2) + d0 * 2) = kraw[it];
        if (!QUADS || 16 * it + quad < keep || 16 * it + quad + 4 > hi) {            // (uniform: a quad at an end of the rows that stay)
          const uint32_t rw[4] = {vraw[it].x, vraw[it].y, vraw[it].z, vraw[it].w};
          int dw, bit;
          v_field(row & 31, d0, 16, &dw, &bit);
          uint16_t* blk16 = reinterpret_cast<uint16_t*>(vr + (row >> 5) * (512 * 16));
#pragma unroll
          for (int e = 0; e < 8; ++e) blk16[(dw + 4 * e) * 2 + (bit >> 4)] = (uint16_t)(rw[e >> 1] >> (16 * (e & 1)));
        }
      }
    } else if (complete && row < lo) {                     // older tokens of the block being flushed
      kraw[it] = *reinterpret_cast<const uint4*>(kr + row * (kHeadDim * 2) + d0 * 2);
      uint32_t code[8];
      value_patterns8(vr, row, d0, code);
      vraw[it] = make_uint4(code[0] | (code[1] << 16), code[2] | (code[3] << 16), code[4] | (code[5] << 16),
                            code[6] | (code[7] << 16));
    }
  }
  if (!complete) return;                                   // uniform over the workgroup

  // rows of all four planes are addressed by the block's first token in plane order (a block never straddles a page)
  const int64_t tv0 = virtual_token(g, c.page_table, b, h, (int64_t)blk * RLT);
  uint8_t* kc = (uint8_t*)c.k_codes;
  uint32_t* km_tok = (uint32_t*)c.k_meta;                                // token-wise keys: entries by token and group
  uint32_t* vm = (uint32_t*)c.v_meta;

  if constexpr (KTOK) {
    // ---- keys token-wise: every row on its own, exactly as quantize_append_kernel does it
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int64_t t = tv0 + rg + 16 * it;
      const uint32_t rw[4] = {kraw[it].x, kraw[it].y, kraw[it].z, kraw[it].w};
      float xk[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) xk[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), BF);
      if (g.rotate_k) rotate8(xk, lane16, rot_sign_bits(g.signs_k, lane16));
      uint32_t kcodes[8];
      uint16_t S, Z;
      const int lpg = g.g_k >> 3;
      quantize8(xk, BK, lpg, kcodes, &S, &Z);
      if ((lane16 & (lpg - 1)) == 0)
        __builtin_nontemporal_store((uint32_t)S | ((uint32_t)Z << 16), km_tok + meta_index(t, lane16 >> lpg_shift(lpg), g.ng_k));
      store_key_codes<BK, true>(kc + t * (16 * BK), lane16, kcodes);
    }
  } else {
    // ---- keys: minimum and maximum of every channel over the rows of each group.  A thread's rows rg + 16 it fall
    // into group it / gi (gi = seq_g / 16 of its rows in a row per group); within a group: this thread's rows, the 4 row
    // groups of its wavefront by two swaps, the 4 wavefronts through LDS.
    const int gi = g.seq_g >> 4;                         // 2, 4 or 8 (uniform)
    uint32_t* km = (uint32_t*)c.k_meta + (tv0 / g.seq_g) * kHeadDim;     // the block's first group: 128 entries each
    const uint32_t signs = rot_sign_bits(g.signs_k, lane16);
    float x[NIT][8];
    float mn[8], mx[8];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const uint32_t rw[4] = {kraw[it].x, kraw[it].y, kraw[it].z, kraw[it].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) x[it][e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), BF);
      // rotated keys: the block's rows are quantized as R k (the buffer keeps the input rows; the 16 lanes of a row are
      // neighbours in one wavefront, and the whole workgroup is here)
      if (g.rotate_k) rotate8(x[it], lane16, signs);
      const bool first = (it & (gi - 1)) == 0, last = ((it + 1) & (gi - 1)) == 0;
      if (first) {                                       // (uniform)
#pragma unroll
        for (int e = 0; e < 8; ++e) mn[e] = mx[e] = x[it][e];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) { mn[e] = min2f(mn[e], x[it][e]); mx[e] = max2f(mx[e], x[it][e]); }
      }
      if (last) {                                        // (uniform)
        const int grp = it / gi;
        float4 w[4];
        float* wf = reinterpret_cast<float*>(w);
#pragma unroll
        for (int e = 0; e < 8; ++e) { wf[e] = rows_min(mn[e]); wf[8 + e] = rows_max(mx[e]); }
        if ((rg & 3) == 0) {
          float4* pn = reinterpret_cast<float4*>(&s_mn[grp][tid >> 6][d0]);
          float4* px = reinterpret_cast<float4*>(&s_mx[grp][tid >> 6][d0]);
          pn[0] = w[0]; pn[1] = w[1]; px[0] = w[2]; px[1] = w[3];
        }
      }
    }
    __syncthreads();
    const float levels = (float)((1 << BK) - 1);
    const int n_grp = RLT / g.seq_g;
    for (int i = tid; i < n_grp * kHeadDim; i += 256) {  // one thread per channel and group
      const int grp = i >> 7, d = i & (kHeadDim - 1);
      const float lo_v = min2f(min2f(s_mn[grp][0][d], s_mn[grp][1][d]), min2f(s_mn[grp][2][d], s_mn[grp][3][d]));
      const float hi_v = max2f(max2f(s_mx[grp][0][d], s_mx[grp][1][d]), max2f(s_mx[grp][2][d], s_mx[grp][3][d]));
      uint16_t S, Z;
      group_scale_zero(lo_v, hi_v, BK, &S, &Z);
      __builtin_nontemporal_store((uint32_t)S | ((uint32_t)Z << 16), km + i);
      const float sc = widen16(S, false);
      s_zero[grp][d] = widen16(Z, false);
      s_rcp[grp][d] = sc == 0.0f ? 0.0f : rcp_scale(sc);  // (a scale of 0: every code is 0)
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int grp = it / gi;
      const float4* pz = reinterpret_cast<const float4*>(&s_zero[grp][d0]);
      const float4* pr = reinterpret_cast<const float4*>(&s_rcp[grp][d0]);
      const float4 z0 = pz[0], z1 = pz[1], r0 = pr[0], r1 = pr[1];
      const float z[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
      const float rcp[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
      uint32_t codes[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) codes[e] = group_code(x[it][e], z[e], rcp[e], levels);
      store_key_codes<BK, true>(kc + (tv0 + rg + 16 * it) * (16 * BK), lane16, codes);
    }
  }

  // ---- values: token-wise, as in quantize_append_kernel for a full span, one span of kSpan tokens after the other
#pragma unroll
  for (int sp = 0; sp < RLT / kSpan; ++sp) {
    if (sp) __syncthreads();                             // (the staging area is reused)
#pragma unroll
    for (int k = 0; k < kSpan / 16; ++k) {
      const int it = sp * (kSpan / 16) + k;
      const int row = rg + 16 * k;                       // row inside the span
      const int64_t t = tv0 + sp * kSpan + row;
      const uint32_t rw[4] = {vraw[it].x, vraw[it].y, vraw[it].z, vraw[it].w};
      float xv[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) xv[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), BF);
      uint32_t vcodes[8];
      uint16_t S, Z;
      const int lpg = g.g_v >> 3;
      quantize8(xv, BV, lpg, vcodes, &S, &Z);
      if ((lane16 & (lpg - 1)) == 0) {
        __builtin_nontemporal_store((uint32_t)S | ((uint32_t)Z << 16), vm + meta_index(t, lane16 >> lpg_shift(lpg), g.ng_v));
        note_value_scale(c.v_scale_exp + bh, S);
      }
      stage_value_row<BV>(vstage, row, d0, vcodes);
    }
    __syncthreads();
    store_value_span<BV, kSpan, true>((uint32_t*)c.v_codes + ((tv0 + sp * kSpan) >> 5) * (128 * BV), vstage, tid, 0, kSpan);
  }
}

}  // namespace

namespace {
// Whether the input rows are read by streaming loads.  An input of up to 256 MiB, the size of the last-level cache, may lie
// there, where the kernel before left it, and streaming loads do not find it: 16 x 8 heads x 2048 tokens, K4V2 channel-wise, on
// the same input 83.7 us with them and 70.3 without (on three inputs in turn, which the cache does not hold, 84.3 and
// 83.9); 48 x 8 x 1000 81.8 and 64.6 (82.3 and 81.4).  Larger inputs gain from them: 8 x 8 x 8229, rotated, 76.8 and 78.5;
// so do launches of up to two workgroups per unit, which all ask at once: 4 x 8 x 1024 on three inputs in turn 14.5 and
// 15.1 (on the same one 13.9 and 13.4).
constexpr int64_t kCacheBytes = (int64_t)256 << 20;
bool stream_in(const Geom& g, int32_t n_new, dim3 grid) {
  const int64_t bytes = (int64_t)g.batch * g.kv_heads * n_new * (2 * kHeadDim * 2);
  return bytes > kCacheBytes || (int64_t)grid.x * grid.y <= 2 * device_compute_units();
}
// pos_arr != nullptr: one token per sequence at pos_arr[b] (then pos and n_new are 0 and 1)
template <int BK, int BV, bool STREAM_IN>
void launch_sa_in(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb, int64_t sh,
                  int64_t st, int32_t pos, int32_t n_new, const int32_t* pos_arr, int32_t max_pos, dim3 grid, hipStream_t stream) {
  const bool bf = in_dtype == KVQ_BF16, ktok = g.axis_k != KVQ_AXIS_SEQ;
#define KVQ_SA_LAUNCH(BF_, KTOK_, RL_)                                                                                     \
  hipLaunchKernelGGL((seq_append_kernel<BK, BV, BF_, KTOK_, RL_, STREAM_IN, KVQ_QUADS>), grid, dim3(256), 0, stream, g, c,            \
                     (const uint16_t*)k_new, (const uint16_t*)v_new, sb, sh, st, pos, n_new, pos_arr, max_pos)
  if (ktok) { if (bf) KVQ_SA_LAUNCH(true, true, 64); else KVQ_SA_LAUNCH(false, true, 64); }
  else if (g.resid == 128) { if (bf) KVQ_SA_LAUNCH(true, false, 128); else KVQ_SA_LAUNCH(false, false, 128); }
  else { if (bf) KVQ_SA_LAUNCH(true, false, 64); else KVQ_SA_LAUNCH(false, false, 64); }
#undef KVQ_SA_LAUNCH
}
template <int BK, int BV>
hipError_t launch_sa(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb,
                     int64_t sh, int64_t st, int32_t pos, int32_t n_new, const int32_t* pos_arr, int32_t max_pos,
                     hipStream_t stream) {
  const int first = pos / g.resid, last = (pos + n_new - 1) / g.resid;
  const dim3 grid(last - first + 1, g.batch * g.kv_heads);
  if (stream_in(g, n_new, grid)) launch_sa_in<BK, BV, true>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, grid, stream);
  else launch_sa_in<BK, BV, false>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, grid, stream);
  return hipGetLastError();
}
template <int BK>
hipError_t launch_sak(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb,
                      int64_t sh, int64_t st, int32_t pos, int32_t n_new, const int32_t* pos_arr, int32_t max_pos,
                      hipStream_t stream) {
  switch (g.bits_v) {
    case 1: return launch_sa<BK, 1>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 2: return launch_sa<BK, 2>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 3: return launch_sa<BK, 3>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 4: return launch_sa<BK, 4>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 6: return launch_sa<BK, 6>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 8: return launch_sa<BK, 8>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
  }
  return hipErrorInvalidValue;
}
hipError_t launch_sa_bits(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb,
                          int64_t sh, int64_t st, int32_t pos, int32_t n_new, const int32_t* pos_arr, int32_t max_pos,
                          hipStream_t stream) {
  switch (g.bits_k) {
    case 1: return launch_sak<1>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 2: return launch_sak<2>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 3: return launch_sak<3>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 6: return launch_sak<6>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 4: return launch_sak<4>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
    case 8: return launch_sak<8>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, pos_arr, max_pos, stream);
  }
  return hipErrorInvalidValue;
}
}  // namespace

#ifdef KVQ_SA_QUADS
hipError_t launch_sa_quads(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb, int64_t sh,
                           int64_t st, int32_t pos, int32_t n_new, hipStream_t stream) {
  return launch_sa_bits(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, nullptr, 0, stream);
}
#else
hipError_t launch_sa_quads(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb, int64_t sh,
                           int64_t st, int32_t pos, int32_t n_new, hipStream_t stream);

// Whether value patterns leave four tokens at a time (store_value_quads): in launches of two workgroups per unit and more always; in
// smaller ones, which end with the slowest block, where a block that is quantized stores a quarter of the buffer or more as well, and
// where none is quantized.  With less, the transposition's code costs the launch 0.1 to 0.4 us.  Stored one by one and so, 64-token
// buffers, 8 kv heads, by sequences x tokens: 2 x 700 (4 tokens in the last quantized block) 6.1 us and 6 % more, 4 x 440 (8) 6.6 and 4 % more, 3 x 565 (11) 6.6
// and 2 % more, 1 x 1900 (20) 7.0 and 6 % less, 3 x 900 (60) 10.1 and 16 % less, 8 x 60 (none) 5.4 and 42 % less; 512 workgroups and more 0 to 45 % less.
// Where the blocks of a sequence are a multiple of 8, the last ones of all sequences share a part of the chip, and it pays from 24 of them and
// more than one workgroup per unit on: 3 x 1012 9.1 us and 10 % less, 5 x 500 9.4 and 12 % less, 2 x 1524 3 % more, 4 x 500 (256 workgroups) 2 % more.
bool stores_quads(const Geom& g, int32_t pos, int32_t n_new) {
  const int32_t first = pos / g.resid, end = pos + n_new, tail = end % g.resid;
  if (n_new < 4) return false;
  const int64_t streams = g.batch * g.kv_heads, blocks = (end - 1) / g.resid - first + 1;
  if (blocks * streams >= 2 * device_compute_units()) return true;
  if (blocks % 8 == 0 && streams >= 24 && blocks * streams > device_compute_units()) return true;
  const bool quantizes = end / g.resid > first;
  const int32_t stored = n_new < g.resid - tail ? n_new : g.resid - tail;      // by the last block that is quantized
  return !quantizes || 4 * stored >= g.resid;
}

hipError_t launch_seq_append_one(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype,
                                 int64_t sb, int64_t sh, const int32_t* pos_arr, int32_t max_pos, hipStream_t stream) {
  return launch_sa_bits(g, c, k_new, v_new, in_dtype, sb, sh, kHeadDim, 0, 1, pos_arr, max_pos, stream);
}

hipError_t launch_seq_append(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype,
                             int64_t sb, int64_t sh, int64_t st, int32_t pos, int32_t n_new, hipStream_t stream) {
  if (n_new == 0) return hipSuccess;
  // A first block that starts inside the residual buffer reads its older rows from there, while the workgroups of the
  // call's last tokens (as many as the buffer has slots) overwrite those slots: when the call goes on beyond that block, the block gets a launch of
  // its own and the rest follows in stream order.
  const int32_t first_end = (pos / g.resid + 1) * g.resid;
  if (pos % g.resid != 0 && pos + n_new > first_end) {
    const int32_t n1 = first_end - pos;
    hipError_t e = launch_seq_append(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n1, stream);
    if (e != hipSuccess) return e;
    return launch_seq_append(g, c, (const uint16_t*)k_new + (int64_t)n1 * st, (const uint16_t*)v_new + (int64_t)n1 * st,
                             in_dtype, sb, sh, st, first_end, n_new - n1, stream);
  }
  if (stores_quads(g, pos, n_new)) return launch_sa_quads(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
  return launch_sa_bits(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, nullptr, 0, stream);
}
#endif

}  // namespace kvq
