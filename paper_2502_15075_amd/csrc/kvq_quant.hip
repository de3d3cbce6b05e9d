// Quantize-append kernel for token-wise groups, and the quantizer's self-test (gfx950).
//
// The quantizer is the b-bit uniform scalar quantizer of App. B ("Preliminaries": scale factor,
// round, clip, reconstruct) of arXiv 2502.15075 in its group-wise asymmetric min-max form; the
// exact arithmetic is stated in kvq.h.  Codes and scale/zero bytes must be identical on every
// machine, so this file is compiled with floating-point contraction off and every operation
// below is a single IEEE binary32 operation (hipcc's default division is correctly rounded).
#include "kvq_stage.h"

namespace kvq {
namespace {

// One workgroup = `chain` consecutive spans of SPAN tokens (a multiple of 32: whole blocks of value codes) of one (b,h)
// stream, restricted to the new tokens in them.  The rows of the next span are loaded before the current one is
// quantized, so that a workgroup has loads in flight while it computes (with one span per workgroup the kernel waits on
// memory latency: 8 workgroups per compute unit do not keep enough bytes in flight on their own).  No load is
// conditional -- rows outside the new tokens re-read a row inside them, and the load "after the last span" is
// collapsed onto 16 bytes -- so that the compiler can count the loads in flight behind the ones it waits for (the last
// span peeled out of the loop instead, with nothing loaded behind it, costs 20 registers and 7 % of the rate).
template <int BK, int BV, bool BF, int SPAN>
__global__ __launch_bounds__(256) void quantize_append_kernel(Geom g, kvq_cache c, const uint16_t* __restrict__ k_new,
                                                              const uint16_t* __restrict__ v_new, int64_t sb, int64_t sh,
                                                              int64_t st, int32_t pos, int32_t n_new, int32_t chain) {
  constexpr int kSpan = SPAN;                      // (shadows the 64-token span of kvq_stage.h)
  constexpr int NR = SPAN / 16;                    // rows per thread and span
  __shared__ __attribute__((aligned(16))) uint8_t vstage[stage_total<BV, SPAN>()];
  const int tid = threadIdx.x;
  const int bh = blockIdx.y;
  const int b = bh / g.kv_heads, h = bh % g.kv_heads;
  const int lane16 = tid & 15;
  const int d0 = lane16 * 8;
  const int lpg_k = g.g_k >> 3, lpg_v = g.g_v >> 3;                  // lanes per group
  const int km_step = 16 * g.ng_k, vm_step = 16 * g.ng_v;
  const int blk_first = pos / kSpan + blockIdx.x * chain;
  const int blk_end = min(blk_first + chain, (pos + n_new - 1) / kSpan + 1);     // (the grid leaves no workgroup empty)
  const int64_t in_base = (int64_t)b * sb + (int64_t)h * sh;

  // the rows (tid/16) + 16*it of span blk; `live` = 0 collapses all loads onto the first 16 bytes of the span's first
  // new row
  auto load_span = [&](int blk, uint32_t live, uint4 (&kraw)[NR], uint4 (&vraw)[NR]) {
    const int lo = max(pos, blk * kSpan) - blk * kSpan;
    const int hi = min(pos + n_new, (blk + 1) * kSpan) - blk * kSpan;
#pragma unroll
    for (int it = 0; it < NR; ++it) {
      const int row = min(max((tid >> 4) + 16 * it, lo), hi - 1);
      const int64_t first_row = (int64_t)blk * kSpan + lo - pos;
      const int64_t src = in_base + first_row * st + (((int64_t)(row - lo) * st + d0) & (int64_t)(int32_t)live);
      kraw[it] = load_stream16(k_new + src);       // (streaming: the input rows are read once)
      vraw[it] = load_stream16(v_new + src);
    }
  };

  // (formed once: inside the loop over the spans they cost a bulk append 2 %, also one that does not rotate:
  // 64 x 8 heads x 2048 tokens K4V2 246.7 us against 242.0)
  const uint32_t signs_k = rot_sign_bits(g.signs_k, lane16), signs_v = rot_sign_bits(g.signs_v, lane16);
  uint4 kraw[NR], vraw[NR], knext[NR], vnext[NR];
  load_span(blk_first, ~0u, kraw, vraw);
  for (int blk = blk_first; blk < blk_end; ++blk) {
    const bool more = blk + 1 < blk_end;           // uniform
    load_span(more ? blk + 1 : blk, more ? ~0u : 0u, knext, vnext);
    const int lo = max(pos, blk * kSpan) - blk * kSpan;
    const int hi = min(pos + n_new, (blk + 1) * kSpan) - blk * kSpan;
    // rows of all four planes are addressed by the span's first token in plane order (a span never straddles a page)
    const int64_t tv0 = virtual_token(g, c.page_table, b, h, (int64_t)blk * kSpan);
    uint32_t* vc = (uint32_t*)c.v_codes + (tv0 >> 5) * (128 * BV);
    // tv0 is a multiple of 32 (of the page size when paged), so row (tid/16) + 16*it sits at position tid/16 of the
    // span's it-th slab of 16 tokens in the scale/zero planes: one address per thread, a uniform stride per it
    uint8_t* kc = (uint8_t*)c.k_codes + (tv0 + (tid >> 4)) * (BK == 16 ? 256 : 16 * BK);
    uint32_t* km = (uint32_t*)c.k_meta + meta_index(tv0 + (tid >> 4), lane16 >> lpg_shift(lpg_k), g.ng_k);
    uint32_t* vm = (uint32_t*)c.v_meta + meta_index(tv0 + (tid >> 4), lane16 >> lpg_shift(lpg_v), g.ng_v);
#pragma unroll
    for (int it = 0; it < NR; ++it) {
      const int row = (tid >> 4) + 16 * it;
      if (row < lo || row >= hi) continue;         // whole 16-lane rows take the same branch
      // ---- keys: row-major codes
      {
        const uint4 raw = kraw[it];
        const uint32_t rw[4] = {raw.x, raw.y, raw.z, raw.w};
        if (BK == 16) {
          store_stream16(kc + it * (16 * 256) + d0 * 2, raw);
        } else {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), BF);
          if (g.rotate_k) rotate8(x, lane16, signs_k);   // whole 16-lane rows are here together
          uint32_t codes[8];
          uint16_t S, Z;
          quantize8(x, BK, lpg_k, codes, &S, &Z);
          if ((lane16 & (lpg_k - 1)) == 0) __builtin_nontemporal_store((uint32_t)S | ((uint32_t)Z << 16), km + it * km_step);
          store_key_codes<BK, true>(kc + it * (16 * 16 * BK), lane16, codes);
        }
      }
      // ---- values: scale/zero straight to memory, codes to their place in the staged words
      {
        const uint4 raw = vraw[it];
        const uint32_t rw[4] = {raw.x, raw.y, raw.z, raw.w};
        uint32_t codes[8];
        if (BV == 16) {
#pragma unroll
          for (int e = 0; e < 8; ++e) codes[e] = (rw[e >> 1] >> (16 * (e & 1))) & 0xFFFFu;
        } else {
          float x[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) x[e] = widen16((uint16_t)(rw[e >> 1] >> (16 * (e & 1))), BF);
          if (g.rotate_v) rotate8(x, lane16, signs_v);
          uint16_t S, Z;
          quantize8(x, BV, lpg_v, codes, &S, &Z);
          if ((lane16 & (lpg_v - 1)) == 0) {
            __builtin_nontemporal_store((uint32_t)S | ((uint32_t)Z << 16), vm + it * vm_step);
            note_value_scale(c.v_scale_exp + bh, S);
          }
        }
        stage_value_row<BV, SPAN>(vstage, row, d0, codes);
      }
    }
    __syncthreads();
    store_value_span<BV, SPAN, true>(vc, vstage, tid, lo, hi);
    if (more) __syncthreads();                     // (the staging area is reused by the next span)
#pragma unroll
    for (int it = 0; it < NR; ++it) { kraw[it] = knext[it]; vraw[it] = vnext[it]; }
  }
}

// Checks the quantizer's fast divisions on the device it runs on: counters[0] counts the binary16 scales whose fast
// reciprocal differs from IEEE division (all 31743 positive finite patterns), counters[1] the sampled quotients
// (2^24 numerators per level count, spread over the binary32 exponent range) that differ.
__global__ __launch_bounds__(256) void selftest_quantizer_kernel(uint32_t* counters) {
#pragma clang fp contract(off)
  const uint32_t u = blockIdx.x * 256 + threadIdx.x;          // 0 .. 65535
  uint32_t bad_rcp = 0, bad_div = 0;
  if (u >= 1 && u < 0x7C00) {
    const float s = widen16((uint16_t)u, false);
    if (rcp_scale(s) != 1.0f / s) bad_rcp = 1;
  }
  const int widths[6] = {1, 2, 3, 4, 6, 8};
  for (uint32_t i = 0; i < 256; ++i) {
    const uint32_t bits = (uint32_t)(((uint64_t)(u * 256u + i) * 0x7F800000ull) >> 24);   // every 128th binary32 >= 0
    const float x = __uint_as_float(bits);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      const float levels = (float)((1 << widths[k]) - 1);
      const float fast = div_levels(x, levels, inv_levels(widths[k])), exact = x / levels;
      if (fast != exact || f32_to_f16_bits(fast) != f32_to_f16_bits(exact)) ++bad_div;
    }
  }
  if (bad_rcp) atomicAdd(counters, bad_rcp);
  if (bad_div) atomicAdd(counters + 1, bad_div);
}

__global__ __launch_bounds__(64) void zero_u32_kernel(uint32_t* p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0u;
}

}  // namespace

namespace {
template <int BK, int BV>
hipError_t launch_q(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb,
                    int64_t sh, int64_t st, int32_t pos, int32_t n_new, hipStream_t stream) {
  // one workgroup per 32-token span (one block of value codes): against 64-token spans this doubles the workgroups of a
  // small call (a 2048-token chunk of one sequence: 6.5 instead of 7.9 us) and costs a large one nothing
  constexpr int kQSpan = 32;
  const int first = pos / kQSpan, last = (pos + n_new - 1) / kQSpan;
  // spans per workgroup: 4 in a row (each loaded while the one before is quantized) when that still leaves every
  // compute unit many rounds of workgroups (the 70B layer's bulk fill: 5.6 against 5.15 TB/s; 2 or 8 in a row
  // measure 5.4), one for smaller calls, which need their workgroups side by side
  const int64_t spans = (int64_t)(last - first + 1) * g.batch * g.kv_heads;
  const int chain = spans >= 65536 ? 4 : 1;
  dim3 grid((last - first + chain) / chain, g.batch * g.kv_heads);
  if (in_dtype == KVQ_BF16)
    hipLaunchKernelGGL((quantize_append_kernel<BK, BV, true, kQSpan>), grid, dim3(256), 0, stream, g, c, (const uint16_t*)k_new,
                       (const uint16_t*)v_new, sb, sh, st, pos, n_new, chain);
  else
    hipLaunchKernelGGL((quantize_append_kernel<BK, BV, false, kQSpan>), grid, dim3(256), 0, stream, g, c, (const uint16_t*)k_new,
                       (const uint16_t*)v_new, sb, sh, st, pos, n_new, chain);
  return hipGetLastError();
}
template <int BK>
hipError_t launch_qk(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype, int64_t sb,
                     int64_t sh, int64_t st, int32_t pos, int32_t n_new, hipStream_t stream) {
  switch (g.bits_v) {
    case 1: return launch_q<BK, 1>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 2: return launch_q<BK, 2>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 3: return launch_q<BK, 3>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 4: return launch_q<BK, 4>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 6: return launch_q<BK, 6>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 8: return launch_q<BK, 8>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 16: return launch_q<BK, 16>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
  }
  return hipErrorInvalidValue;
}
}  // namespace

hipError_t launch_quantize_append(const Geom& g, const kvq_cache& c, const void* k_new, const void* v_new, int in_dtype,
                                  int64_t sb, int64_t sh, int64_t st, int32_t pos, int32_t n_new, hipStream_t stream) {
  if (n_new == 0) return hipSuccess;
  switch (g.bits_k) {
    case 1: return launch_qk<1>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 2: return launch_qk<2>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 3: return launch_qk<3>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 4: return launch_qk<4>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 6: return launch_qk<6>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 8: return launch_qk<8>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
    case 16: return launch_qk<16>(g, c, k_new, v_new, in_dtype, sb, sh, st, pos, n_new, stream);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_selftest_quantizer(uint32_t* counters, hipStream_t stream) {
  hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, stream, counters, 2);
  hipLaunchKernelGGL(selftest_quantizer_kernel, dim3(256), dim3(256), 0, stream, counters);
  return hipGetLastError();
}

}  // namespace kvq
