"""What the framework is timed on: the calls that a program with a quantized key/value cache makes, over the range of
sizes, cache formats and data types that such programs use.

A case is a dict of plain values:
  call      "step"    the loop body of chunk-wise generation: the newest cached chunk is (re)written with
                      kvq_quantize_append, then the current chunk's queries attend to the cached window and to the
                      unquantized current keys (kvq_chunk_attention)
            "attend"  kvq_chunk_attention alone: a generator attends several times to a window between two appends
            "prefill" kvq_chunk_attention_ex: grouped query heads, causal current block, a quantized prefix
            "append"  kvq_quantize_append alone
  heads     key/value heads;  ratio: query heads per key/value head
  dim, bits, io ("bf16" / "fp32"), meta ("fp32" / "fp8"), group (channels per pair), axis ("token" / "channel")
  chunk     tokens of an appended chunk
  rows      query rows;  current: unquantized current keys;  cached: cached tokens attended to
  ragged    tokens that the window has slid past: it starts inside the ring, and inside a tile where that is odd
"""
from __future__ import annotations

import math

import torch

from paper_2605_26266_amd import binding as kvq

DEV = "cuda:0"


def _case(name, call, heads, dim, bits, chunk, rows, current, cached, io="bf16", meta="fp32", group=None, axis="token",
          ratio=1, ragged=0):
    c = dict(call=call, heads=heads, ratio=ratio, dim=dim, bits=bits, io=io, meta=meta, group=dim if group is None else group,
             axis=axis, chunk=chunk, rows=rows, current=current, cached=cached, ragged=ragged)
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest step: one head, head_dim 64, fp32 tensors, a few hundred keys.  Launches and latency.
        _case("tiny_step_fp32", "step", 1, 64, 2, 64, 64, 64, 256, io="fp32"),
        # A small generator: 8 heads, 1024-token chunks, four chunks cached; the window has slid over the ring.
        _case("small_step", "step", 8, 128, 2, 1024, 1024, 1024, 4096, ragged=1024),
        # The same with keys quantized per channel and appended block.
        _case("small_step_channel", "step", 8, 128, 2, 1024, 1024, 1024, 4096, axis="channel"),
        # The last token of a prompt (or the next one) against a quantized prefix: grouped heads, one query row.
        _case("prefill_tail", "prefill", 8, 128, 2, 2048, 1, 64, 8192, meta="fp8", group=32, ratio=4),
        # One block of a chunked prefill behind the same prefix, 4-bit codes with groups of 64.
        _case("prefill_block", "prefill", 8, 128, 4, 2048, 1000, 1000, 8192, meta="fp8", group=64, ratio=4),
        # head_dim 64 with BF16 tensors, odd sizes.
        _case("dim64_attend", "attend", 12, 64, 2, 500, 500, 500, 1500),
        # The mid-size generator: 24 heads, 4680-token chunks (not a multiple of any tile), six cached chunks, with
        # 2-bit and 4-bit codes and with the format the method is published with (groups of 32, FP8/BF16 metadata).
        _case("mid_step", "step", 24, 128, 2, 4680, 4680, 4680, 28080),
        _case("mid_attend_int4", "attend", 24, 128, 4, 4680, 4680, 4680, 28080),
        _case("mid_step_group32", "step", 24, 128, 2, 4680, 4680, 4680, 28080, meta="fp8", group=32, ragged=4680),
        # The largest step: 48 heads, 4096-token chunks, sixteen cached.
        _case("large_step", "step", 48, 128, 2, 4096, 4096, 4096, 65536),
        # Appends alone: a large chunk, and a chunk of a size that no tile divides, begun inside a tile.
        _case("append_large", "append", 48, 128, 2, 4096, 0, 0, 8192),
        _case("append_group32", "append", 24, 128, 2, 4680, 0, 0, 9360, meta="fp8", group=32, ragged=17),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_FORMATS = [("fp32", 128, "token"), ("fp32", 128, "token"), ("fp8", 32, "token"), ("fp8", 64, "token"),
            ("fp8", 128, "token"), ("fp32", 128, "channel")]


def draw(rng):
    call = rng.choice(["step", "step", "step", "attend", "prefill", "prefill", "append", "vector"])
    bits = rng.choice([2, 2, 4])
    meta, group, axis = rng.choice(_FORMATS)
    ragged = rng.choice([0, 0, 32 * rng.randint(1, 40), rng.randint(1, 200)])
    if call == "append":
        heads, chunk = rng.randint(1, 48), _log_int(rng, 64, 4680)
        if axis == "channel":
            meta, group, axis = "fp8", 32, "token"
        return _case(None, "append", heads, 128, bits, chunk, 0, 0, 2 * chunk, meta=meta, group=group, axis=axis, ragged=ragged)
    if call == "prefill":     # a block or the tail of a prompt behind a quantized prefix
        heads, ratio = rng.choice([2, 4, 8]), rng.choice([1, 3, 4, 8])
        cached, current = _log_int(rng, 500, 16384), _log_int(rng, 64, 2048)
        rows = rng.choice([1, rng.randint(2, 64), current])
        if axis == "channel":
            meta, group, axis = "fp32", 128, "token"
        return _case(None, "prefill", heads, 128, bits, 2048, min(rows, current), current, cached, meta=meta, group=group,
                     ratio=ratio, ragged=ragged)
    if call == "vector":      # fp32 tensors or head_dim 64
        io, dim = rng.choice([("fp32", 64), ("fp32", 128), ("bf16", 64)])
        heads, chunk = rng.randint(1, 12), _log_int(rng, 64, 600)
        cached = min(chunk * rng.randint(1, 6), int(4e9 / (4 * heads * chunk * dim)))
        meta, group = rng.choice([("fp32", dim), ("fp32", dim), ("fp8", 32)])
        return _case(None, rng.choice(["step", "attend"]), heads, dim, bits, min(chunk, cached), chunk, chunk, cached, io=io,
                     meta=meta, group=group, ragged=ragged)
    heads, chunk = _log_int(rng, 1, 48), _log_int(rng, 64, 4680)
    cached = chunk * _log_int(rng, 1, 32)
    while 4.0 * heads * chunk * (cached + chunk) * 128 > 3.5e12:
        cached -= chunk
    return _case(None, call, heads, 128, bits, chunk, chunk, chunk, max(cached, chunk), meta=meta, group=group, axis=axis,
                 ragged=ragged)


def _inputs(case, seed):
    """Yields ("slid", k, v) for the tokens the window has slid past, ("chunk", k, v) for each cached chunk, ("new", k, v)
    for the chunk that run() appends and ("query", q, k_cur, v_cur), in this order, where the case has them."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    heads, dim, io = case["heads"], case["dim"], torch.bfloat16 if case["io"] == "bf16" else torch.float32

    def normal(tokens, n_heads):
        return torch.randn((tokens, n_heads, dim), generator=gen, device=DEV).to(torch.bfloat16)

    # Keys carry a few channels much larger than the rest (the same ones for every token of a head).
    gain = torch.ones((heads, dim), device=DEV)
    for h in range(heads):
        gain[h, torch.randperm(dim, generator=gen, device=DEV)[: max(1, round(0.02 * dim))]] = 10.0

    def kv(tokens):   # values that BF16 holds, in the tensors' type
        return (normal(tokens, heads) * gain).to(torch.bfloat16).to(io), normal(tokens, heads).to(io)

    ahead = _ahead(case)
    if case["ragged"] and ahead:       # the window has slid: older tokens came before its first chunk and are gone
        yield ("slid", *kv(case["ragged"]))
    for start in range(0, ahead, case["chunk"]):
        yield ("chunk", *kv(min(case["chunk"], ahead - start)))
    if case["call"] in ("step", "append"):
        yield ("new", *kv(case["chunk"]))
    if case["call"] != "append":
        yield ("query", normal(case["rows"], heads * case["ratio"]).to(io), *kv(case["current"]))


def _ahead(case):   # tokens in the cache before the chunk that run() appends (all of the window where it appends none)
    return case["cached"] - (case["chunk"] if case["call"] in ("step", "append") else 0)


def prepare(case, seed):
    heads, ragged, ahead = case["heads"], case["ragged"], _ahead(case)
    capacity = max(case["cached"] + 64, ragged + min(case["chunk"], ahead))
    cache = kvq.Cache(kvq.make_desc(
        heads, case["dim"], case["bits"], capacity, kvq.KVQ_BF16 if case["io"] == "bf16" else kvq.KVQ_FP32, case["group"], 1,
        kvq.KVQ_META_FP32 if case["meta"] == "fp32" else kvq.KVQ_META_FP8_BF16,
        kvq.KVQ_KEYS_PER_TOKEN if case["axis"] == "token" else kvq.KVQ_KEYS_PER_CHANNEL), DEV)
    cache.storage.zero_()
    state = {"case": case, "cache": cache, "base": ahead}
    slid = 0
    for what, *tensors in _inputs(case, seed):
        if what == "query":
            q, state["k_cur"], state["v_cur"] = tensors
            state.update(q=q, out=torch.empty_like(q))
            state["mass"] = torch.empty((heads * case["ratio"], case["rows"]), dtype=torch.float32, device=DEV)
        elif what == "new":
            state["k"], state["v"] = tensors
        else:
            kvq.kvq_quantize_append(cache, *tensors)
            if what == "chunk" and slid:
                kvq.kvq_cache_evict(cache, slid)
            slid = ragged if what == "slid" else 0
    return state


def run(state):
    cache, call = state["cache"], state["case"]["call"]
    if call in ("step", "append"):
        kvq.kvq_cache_truncate(cache, state["base"])
        kvq.kvq_quantize_append(cache, state["k"], state["v"])
    if call == "append":
        return cache.storage
    attend = kvq.kvq_chunk_attention_ex if call == "prefill" else kvq.kvq_chunk_attention
    options = {"causal": True} if call == "prefill" else {}
    attend(cache, 0, len(cache), state["q"], state["k_cur"], state["v_cur"], state["out"], state["mass"], **options)
    return {"out": state["out"], "mass": state["mass"]}


def work(case):
    heads, dim, elt = case["heads"], case["dim"], 2 if case["io"] == "bf16" else 4
    q_heads = heads * case["ratio"]
    meta = 8 if case["meta"] == "fp32" else 3 * (dim // case["group"])
    packed = dim * case["bits"] / 8 + meta      # of one token, head and tensor
    n_bytes = flops = 0.0
    if case["call"] in ("step", "append"):      # K and V in, codes and metadata out; butterflies and four operations per element
        n_bytes += 2.0 * case["chunk"] * heads * (dim * elt + packed)
        flops += 2.0 * case["chunk"] * heads * dim * (math.log2(dim) + 4)
    if case["call"] != "append":                # Q, current K and V and the packed window in, O and the masses out
        visible = case["current"] - (case["rows"] - 1) / 2 if case["call"] == "prefill" else case["current"]
        n_bytes += 2.0 * q_heads * case["rows"] * dim * elt + 4.0 * q_heads * case["rows"]
        n_bytes += 2.0 * heads * (case["current"] * dim * elt + case["cached"] * packed)
        flops += 4.0 * q_heads * case["rows"] * (case["cached"] + visible) * dim
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    """About four times what the path shows against the same call in 64 bits (worst listed case: bf16 with head_dim 128
    2.5e-3 and 3.5e-2, where probabilities are rounded to 16 bits too; head_dim 64 1.7e-3 and 4e-3, the rounding of the
    output alone; fp32 5.4e-7 and 2.9e-6 with 320 keys, more with thousands)."""
    if case["call"] == "append":
        return "exact"
    if case["io"] == "fp32":
        return {"rel": 1e-5, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.15} if case["dim"] == 128 else {"rel": 7e-3, "max": 2e-2}


def _round_trip(x, bits, group, meta, per_channel, dim):
    """A chunk [tokens][heads][dim] after rotation, quantization and reconstruction, with the steps [tokens][heads][group
    or 1] (all in the rotated basis): asymmetric round-to-nearest over groups of `group` channels of a token, or over the
    chunk's tokens for each channel."""
    levels, norm = 2.0 ** bits - 1.0, dim ** -0.5
    u = x.double() @ _hadamard(dim)
    u = u if per_channel else u.unflatten(2, (dim // group, group))
    axis = 0 if per_channel else 3
    lo, hi = u.amin(axis, keepdim=True), u.amax(axis, keepdim=True)
    lo, hi = torch.where(hi == lo, lo.clamp(max=0), lo), torch.where(hi == lo, hi.clamp(min=0), hi)
    step = (hi - lo) / levels * norm
    if meta == "fp8":          # the smallest E4M3 value that covers the range; the nearest BF16 zero-point
        ulp = torch.exp2(torch.floor(torch.log2(step.clamp(2.0 ** -6, 448.0))) - 3)
        step = torch.ceil(step.clamp(max=448.0) / ulp) * ulp
    inv = torch.where(step > 0, norm / step, torch.zeros_like(step))
    zero = -torch.round(lo * inv)
    if meta == "fp8":
        zero = zero.to(torch.bfloat16).double()
    else:
        step = step.float().double()
    code = (torch.round(u * inv) + zero).clamp(0, levels)
    return ((code - zero) * step).reshape(x.shape), (step if per_channel else step.squeeze(3)).expand(x.shape[0], -1, -1)


def _hadamard(dim):
    h = torch.ones((1, 1), dtype=torch.float64, device=DEV)
    while h.shape[0] < dim:
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, -h], 1)], 0)
    return h


def exact(case, seed):
    """Quantizer and attention in 64 bits: scores of the cached keys less softmax_scale^2 / 24 * sum over groups of
    step^2 * |q of the group|^2, one softmax over cached and current keys.  None for appended bytes."""
    if case["call"] == "append":
        return None
    dim, per_channel = case["dim"], case["axis"] == "channel"
    cached = []
    for what, *tensors in _inputs(case, seed):
        if what == "query":
            q, k_cur, v_cur = tensors
        elif what != "slid":
            k, step = _round_trip(tensors[0], case["bits"], case["group"], case["meta"], per_channel, dim)
            v, _ = _round_trip(tensors[1], case["bits"], case["group"], case["meta"], False, dim)
            cached.append((k.float(), v.float(), step.float()))   # products of a small integer and a stored step
    k_hat, v_hat, step = (torch.cat(t) for t in zip(*cached))
    rows, heads_q, current, scale = case["rows"], case["heads"] * case["ratio"], case["current"], dim ** -0.5
    rot = _hadamard(dim) * scale
    out = torch.empty((rows, heads_q, dim), dtype=torch.float64, device=DEV)
    mass = torch.empty((heads_q, rows), dtype=torch.float64, device=DEV)
    for h in range(heads_q):
        g = h // case["ratio"]
        k_s, v_s, step2 = k_hat[:, g].double(), v_hat[:, g].double(), step[:, g].double() ** 2
        k_r, v_r = k_cur[:, g].double(), v_cur[:, g].double()
        for r in range(0, rows, 1024):
            x = q[r:r + 1024, h].double()
            y = x @ rot
            nu = (y * y).unflatten(1, (step2.shape[1], dim // step2.shape[1])).sum(2)
            s = torch.cat([y @ k_s.T * scale - nu @ step2.T * (scale * scale / 24.0), x @ k_r.T * scale], 1)
            if case["call"] == "prefill":
                row = torch.arange(r, r + x.shape[0], device=DEV)[:, None] + (current - rows)
                s[:, k_s.shape[0]:].masked_fill_(torch.arange(current, device=DEV)[None, :] > row, float("-inf"))
            p = torch.softmax(s, 1)
            out[r:r + 1024, h] = p[:, :k_s.shape[0]] @ v_s @ rot + p[:, k_s.shape[0]:] @ v_r
            mass[h, r:r + 1024] = p[:, :k_s.shape[0]].sum(1)
    return {"out": out, "mass": mass}
