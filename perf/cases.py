"""The calls that a program holding a mixed-precision KV cache makes, as timing cases.

A case names one call of the public binding (paper_2502_15075_amd.kvq) with its sizes and options:

  step      kvq.decode_step         one decode step: the new token's K/V rows go in, the query attends over everything
  ragged    kvq.decode_step_varlen  the same for a serving batch: sequences of different lengths, paged planes
  attn      kvq.decode_attention    attention alone (the unquantized baseline has no fused step; sweeps time this call)
  fill      kvq.quantize_append     prefill: many tokens in one call
  dequant   kvq.dequantize          rows read back (prefill attention over a quantized history, inspection)
  mse       kvq.reconstruction_error  the error studies

Tensors follow the recipe of paper_2502_15075_amd.synth (normal values; keys scaled by 4 with four outlier channels).
"""
import math

import torch

from paper_2502_15075_amd import kvq, synth

D = 128
SCALE = 1.0 / math.sqrt(D)
SIGNS = (0x9E3779B9, 0x7F4A7C15, 0xF39CC060, 0x5CEDC834)      # signs of the randomized Hadamard rotation
DTYPES = {"fp16": torch.float16, "bf16": torch.bfloat16, "fp32": torch.float32}


def _case(kind, batch, q_heads, kv_heads, tokens, dtype="bf16", bits_k=4, bits_v=2, group_k=64, group_v=64, out="fp32",
          axis_seq=False, rotate_k=False, page=0, shortest=0, pos=0, name=None):
    c = dict(kind=kind, batch=batch, q_heads=q_heads, kv_heads=kv_heads, tokens=tokens, dtype=dtype, bits_k=bits_k,
             bits_v=bits_v, group_k=group_k, group_v=group_v, out=out, axis_seq=axis_seq, rotate_k=rotate_k, page=page,
             shortest=shortest, pos=pos)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one sequence of a small model, 1024 tokens, multi-head attention, small groups: launch and latency
        _case("step", 1, 8, 8, 1024, dtype="fp16", group_k=32, group_v=32, name="step_b1_t1024"),
        # a Llama-3-8B layer at an ordinary batch and context
        _case("step", 8, 32, 8, 8192, name="step_8b_t8192"),
        # a Llama-3-70B layer at serving batch and full context
        _case("step", 32, 64, 8, 32768, name="step_70b_t32768"),
        # one long document (an odd length: the last block is partly filled)
        _case("step", 1, 32, 8, 131071, name="step_b1_t131071"),
        # a serving batch: 16 sequences between 600 and 16001 tokens in shuffled 64-token pages, 4-bit keys and values
        _case("ragged", 16, 32, 8, 16001, bits_v=4, page=64, shortest=600, name="step_ragged_paged"),
        # the full-precision baseline that the allocations are compared with
        _case("attn", 8, 32, 8, 32768, bits_k=16, bits_v=16, out="bf16", name="attn_unquantized_t32768"),
        # the per-column back-end with key rotation: channel-wise keys behind the 64-token residual buffer, 37 tokens in it
        _case("step", 8, 32, 8, 8192 + 37, axis_seq=True, rotate_k=True, name="step_channelwise_rotated"),
        # one chunk of a large batch's prefill
        _case("fill", 32, 64, 8, 8192, pos=8192, name="fill_70b_chunk"),
        # one chunk of a single sequence's prefill
        _case("fill", 1, 32, 8, 2048, pos=6144, name="fill_b1_chunk"),
        # prefill into channel-wise keys with rotation (128 blocks and a tail that stays in the buffer)
        _case("fill", 8, 32, 8, 8192 + 37, axis_seq=True, rotate_k=True, name="fill_channelwise_rotated"),
        # the whole cache of an 8B layer read back in the model's type
        _case("dequant", 8, 32, 8, 8192, out="bf16", name="dequantize_8b"),
        # reconstruction error of a whole layer against the rows it was made from
        _case("mse", 8, 32, 8, 32768, name="mse_8b_t32768"),
    ]


ALLOCATIONS = ((4, 2), (4, 2), (2, 4), (4, 4), (8, 8), (2, 2), (3, 2), (8, 4), (4, 1))
HEADS = ((8, 8), (32, 8), (64, 8), (24, 8), (28, 4), (40, 8))


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("step", "step", "step", "ragged", "ragged", "attn", "fill", "fill", "dequant", "mse"))
    q_heads, kv_heads = rng.choice(HEADS)
    bits_k, bits_v = rng.choice(ALLOCATIONS)
    dtype = rng.choice(("bf16", "bf16", "fp16"))
    group_k, group_v = rng.choice((32, 64, 128)), rng.choice((32, 64, 128))
    axis_seq = kind in ("step", "fill") and rng.random() < 0.3
    rotate_k = rng.random() < 0.3
    out, page, shortest, pos = "fp32", 0, 0, 0
    if kind == "attn" and rng.random() < 0.5:
        bits_k = bits_v = 16
        rotate_k = False
    if kind in ("attn", "dequant"):
        out = rng.choice(("fp32", dtype))
    if axis_seq:
        bits_k, bits_v = rng.choice(((4, 2), (2, 4), (4, 4)))
        group_k = rng.choice((64, 64, 128))
    rows = {"step": 3 << 20, "ragged": 3 << 20, "attn": 1 << 20, "fill": 1 << 20, "dequant": 1 << 19, "mse": 3 << 19}[kind]
    batch = _log(rng, 1, 48)
    tokens = _log(rng, 500, max(600, min(131072, rows // (batch * kv_heads))))
    if kind == "ragged":
        batch = max(batch, 4)
        tokens = min(tokens, rows // (batch * kv_heads))
        page = rng.choice((0, 64, 256))
        shortest = max(1, tokens // _log(rng, 2, 40))
    if kind == "fill" and rng.random() < 0.5:
        pos = 0 if axis_seq else rng.randrange(0, 4096)
    return _case(kind, batch, q_heads, kv_heads, tokens, dtype, bits_k, bits_v, group_k, group_v, out, axis_seq, rotate_k,
                 page, shortest, pos)


def _lengths(c):
    """Tokens per sequence of a ragged batch, the longest first: spread evenly between the two ends."""
    n = c["batch"]
    return [c["tokens"] - (c["tokens"] - c["shortest"]) * b // max(1, n - 1) for b in range(n)]


def _layout(c, n_pages=0):
    return kvq.Layout(c["batch"], c["kv_heads"], c["pos"] + c["tokens"], D, c["bits_k"], c["bits_v"], c["group_k"],
                      c["group_v"], axis_k=kvq.AXIS_SEQ if c["axis_seq"] else kvq.AXIS_HEAD_DIM,
                      raw_dtype=kvq.KVQ_BF16 if c["dtype"] == "bf16" else kvq.KVQ_F16, rotate_k=int(c["rotate_k"]),
                      signs_k=SIGNS if c["rotate_k"] else (0, 0, 0, 0), page_tokens=c["page"], n_pages=n_pages)


def _draws(c, seed):
    """K, V [B, H_kv, tokens, D] and q [B, H_q, D].  The queries are scaled (exactly) so that logits spread over a few
    units, as a model's do, and the softmax over many tokens instead of one."""
    K, V, q = synth.make_kvq(seed, c["batch"], c["kv_heads"], c["q_heads"], c["tokens"], D, dtype=DTYPES[c["dtype"]], device="cuda")
    return K, V, q * 0.125


def _order(c, seed):
    """The order in which a ragged batch's lengths are handed to its sequences."""
    g = torch.Generator()
    g.manual_seed(seed)
    return torch.randperm(c["batch"], generator=g).tolist()


def prepare(case, seed):
    c = case
    K, V, q = _draws(c, seed)
    pages = 0 if not c["page"] else c["batch"] * -(-c["tokens"] // c["page"]) + 3
    L = _layout(c, pages)
    cache = kvq.Cache(L, fill=0)
    if pages:
        g = torch.Generator()
        g.manual_seed(seed + 1)
        cache.page_table = torch.randperm(pages, generator=g)[:pages - 3].to(torch.int32).view(c["batch"], -1).contiguous().cuda()
    s = dict(case=c, layout=L, cache=cache)
    kind = c["kind"]
    if kind == "fill":
        s.update(k=K, v=V)
        return s
    if kind in ("dequant", "mse", "attn"):
        kvq.quantize_append(L, cache, K, V, 0)
        if kind == "mse":
            s.update(k=K, v=V, sums=torch.empty(c["batch"], c["kv_heads"], 2, dtype=torch.float64, device="cuda"))
            return s
        if kind == "dequant":
            shape = (c["batch"], c["kv_heads"], c["tokens"], D)
            s.update(k_out=torch.empty(shape, dtype=DTYPES[c["out"]], device="cuda"),
                     v_out=torch.empty(shape, dtype=DTYPES[c["out"]], device="cuda"))
            return s
    s["q"] = q
    s["out"] = torch.empty(c["batch"], c["q_heads"], D, dtype=DTYPES[c["out"]], device="cuda")
    s["workspace"] = torch.empty(max(16, kvq.decode_workspace_bytes(L, c["q_heads"], c["tokens"])), dtype=torch.uint8, device="cuda")
    if kind == "step":
        kvq.quantize_append(L, cache, K[:, :, :-1], V[:, :, :-1], 0)
        s.update(k=K[:, :, -1].contiguous(), v=V[:, :, -1].contiguous())
    elif kind == "ragged":
        kvq.quantize_append(L, cache, K, V, 0)
        lens = _lengths(c)
        pos = torch.tensor([lens[i] - 1 for i in _order(c, seed)], dtype=torch.long, device="cuda")
        at = pos.view(-1, 1, 1, 1).expand(-1, c["kv_heads"], 1, D)
        s.update(k=K.gather(2, at)[:, :, 0].contiguous(), v=V.gather(2, at)[:, :, 0].contiguous(), pos=pos.to(torch.int32))
    return s


def _state(cache):
    return [p for p in cache.planes if p is not None] + [cache.v_scale_exp]


def run(s):
    c, L, cache = s["case"], s["layout"], s["cache"]
    kind = c["kind"]
    if kind == "step":
        kvq.decode_step(L, cache, s["k"], s["v"], c["tokens"] - 1, s["q"], SCALE, s["out"], s["workspace"])
        return [s["out"]] + _state(cache)
    if kind == "ragged":
        kvq.decode_step_varlen(L, cache, s["k"], s["v"], s["pos"], c["tokens"] - 1, s["q"], SCALE, s["out"], s["workspace"])
        return [s["out"]] + _state(cache)
    if kind == "attn":
        return [kvq.decode_attention(L, cache, s["q"], c["tokens"], SCALE, s["out"], s["workspace"])]
    if kind == "fill":
        kvq.quantize_append(L, cache, s["k"], s["v"], c["pos"])
        return _state(cache)
    if kind == "dequant":
        kvq.dequantize(L, cache, 0, c["tokens"], s["k_out"], s["v_out"])
        return [s["k_out"], s["v_out"]]
    return [kvq.reconstruction_error(L, cache, s["k"], s["v"], 0, s["sums"])]


def _row_bytes(c):
    """Packed bytes of one cached token of one head: codes of both tensors and their scale/zero entries."""
    n = 16 * c["bits_k"] + 16 * c["bits_v"]
    if c["bits_k"] != 16:
        n += 4 * D / c["group_k"]                      # (channel-wise: 4 D bytes per group_k tokens, the same)
    if c["bits_v"] != 16:
        n += 4 * D / c["group_v"]
    return n


def work(case):
    c = case
    kind, streams = c["kind"], c["batch"] * c["kv_heads"]
    per_row = _row_bytes(c)
    tokens = sum(_lengths(c)) if kind == "ragged" else c["batch"] * c["tokens"]
    rows = tokens * c["kv_heads"]
    tail = c["tokens"] % (64 if c["group_k"] == 64 else 128) if c["axis_seq"] else 0      # in the residual buffer
    packed = (rows - streams * tail) * per_row + streams * tail * 512
    out_size = 4 if c["out"] == "fp32" else 2
    if kind in ("step", "ragged", "attn"):
        q = c["batch"] * c["q_heads"] * D
        new = 0 if kind == "attn" else streams * (512 + per_row)
        return {"bytes": packed + q * (2 + out_size) + new, "flops": 4.0 * D * tokens * c["q_heads"]}
    if kind == "fill":
        return {"bytes": rows * 512 + packed, "flops": 0}
    if kind == "dequant":
        return {"bytes": packed + rows * 2 * D * out_size, "flops": 0}
    return {"bytes": rows * 512 + packed + streams * 16, "flops": 0}


def tolerance(case):
    c = case
    if c["kind"] in ("fill", "dequant"):               # bytes; one rounding of code * scale + zero
        return "exact"
    if c["kind"] == "mse":                             # differences and eight-channel sums in 32 bits, the rest in 64
        return {"rel": 1e-6}
    # attention: softmax weights times value scales are rounded to 16 bits before the matrix product, queries rotated with
    # the keys too (measured against 64 bits: 2e-4 to 4e-4, and 1.2e-3 over 131071 tokens, where an output is a small
    # difference of many terms); 16-bit outputs are rounded once more (1.6e-3)
    return {"rel": 5e-3 if c["out"] == "fp32" else 8e-3}


# ---- the same in 64 bits, in plain torch ------------------------------------------------------------------------------

def _rotate(x):
    """R x of 128-channel rows in 32 bits: signs, butterflies over strides 1, 2, ..., 64, one scaling."""
    s = torch.tensor([-1.0 if (SIGNS[d // 32] >> (d % 32)) & 1 else 1.0 for d in range(D)], device=x.device)
    x = x * s
    h = 1
    while h < D:
        y = x.view(*x.shape[:-1], D // (2 * h), 2, h)
        x = torch.stack((y[..., 0, :] + y[..., 1, :], y[..., 0, :] - y[..., 1, :]), dim=-2).view(x.shape)
        h *= 2
    return x * torch.tensor(1.0 / math.sqrt(128.0), dtype=torch.float32, device=x.device)


def _unrotate(y):
    """R^T y in 64 bits."""
    s = torch.tensor([-1.0 if (SIGNS[d // 32] >> (d % 32)) & 1 else 1.0 for d in range(D)], dtype=y.dtype, device=y.device)
    h = torch.ones(1, 1, dtype=y.dtype, device=y.device)
    while h.shape[0] < D:
        h = torch.cat((torch.cat((h, h), 1), torch.cat((h, -h), 1)), 0)
    return (y @ h) / math.sqrt(128.0) * s


def _quantized(x, bits, axis):
    """code * scale + zero in 64 bits of 32-bit groups laid along `axis` (the quantizer's own arithmetic is 32-bit)."""
    mn, mx = x.amin(axis, keepdim=True), x.amax(axis, keepdim=True)
    levels = torch.full_like(mn, float((1 << bits) - 1))
    scale, zero = ((mx - mn) / levels).half().float(), mn.half().float()
    codes = torch.round((x - zero) * (torch.ones_like(scale) / scale)).clamp(0.0, float((1 << bits) - 1))
    codes = torch.where(scale == 0, torch.zeros_like(codes), codes)
    return codes.double() * scale.double() + zero.double()


def _rows(c, K, V):
    """Reconstruction of [H, T, D] rows of one sequence in 64 bits, keys in the basis they are stored in; for a cache with
    a residual buffer T is a whole number of its blocks."""
    H, T, _ = K.shape
    K, V = K.float(), V.float()
    if c["rotate_k"]:
        K = _rotate(K)
    if c["bits_k"] == 16:
        K = K.double()
    elif c["axis_seq"]:
        K = _quantized(K.view(H, T // c["group_k"], c["group_k"], D), c["bits_k"], 2).view(H, T, D)
    else:
        K = _quantized(K.view(H, T, D // c["group_k"], c["group_k"]), c["bits_k"], 3).view(H, T, D)
    if c["bits_v"] == 16:
        V = V.double()
    else:
        V = _quantized(V.view(H, T, D // c["group_v"], c["group_v"]), c["bits_v"], 3).view(H, T, D)
    return K, V


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind == "fill":
        return None                                    # bytes: the start's are what they are compared with
    K, V, q = _draws(c, seed)
    B, H, R = c["batch"], c["kv_heads"], c["q_heads"] // c["kv_heads"]
    if kind in ("dequant", "mse"):
        ks, vs = [], []
        for b in range(B):
            Kh, Vh = _rows(c, K[b], V[b])
            if kind == "dequant":
                ks.append(_unrotate(Kh) if c["rotate_k"] else Kh)
                vs.append(Vh)
            else:
                Kr = _rotate(K[b].float()).double() if c["rotate_k"] else K[b].double()
                ks.append((Kr - Kh).square().sum((1, 2)))
                vs.append((V[b].double() - Vh).square().sum((1, 2)))
        return [torch.stack(ks), torch.stack(vs)] if kind == "dequant" else [torch.stack((torch.stack(ks), torch.stack(vs)), -1)]
    lens = [c["tokens"]] * B
    if kind == "ragged":
        spread = _lengths(c)
        lens = [spread[i] for i in _order(c, seed)]
    out = torch.empty(B, c["q_heads"], D, dtype=torch.float64, device=K.device)
    for b in range(B):
        n = lens[b]
        block = max(64, c["group_k"]) if c["axis_seq"] else 1
        flushed = n // block * block
        Kh, Vh = _rows(c, K[b, :, :flushed], V[b, :, :flushed])
        qb = q[b].view(H, R, D)
        stored_q = _rotate(qb.float()).half().double() if c["rotate_k"] else qb.double()     # (rounded once, as documented)
        for h in range(H):
            s = stored_q[h] @ Kh[h].T
            v = Vh[h]
            if flushed < n:
                s = torch.cat((s, qb[h].double() @ K[b, h, flushed:n].double().T), 1)
                v = torch.cat((v, V[b, h, flushed:n].double()), 0)
            out[b, h * R:(h + 1) * R] = torch.softmax(s * SCALE, 1) @ v
    return [out] + [None] * (0 if kind == "attn" else 7 if c["axis_seq"] else 5)      # (the cache's state is bytes)
