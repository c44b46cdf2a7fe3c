"""The fp32 matrix-core attention kernel where its bf16 pieces do not carry the operands (zero-points beyond them, queries, keys
and values near the ends of the fp32 range or not finite) and where the runs of its eight waves are short or change from cached
to current tiles, against the vector kernel, which computes the same expressions in fp32."""
import math

import pytest
import torch

from paper_2605_26266_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (dim, bits, io, meta, group)
FORMATS = [(64, 2, B.KVQ_FP32, B.KVQ_META_FP32, 64), (64, 4, B.KVQ_FP32, B.KVQ_META_FP8_BF16, 32), (64, 4, B.KVQ_BF16, B.KVQ_META_FP32, 64),
           (128, 4, B.KVQ_FP32, B.KVQ_META_FP32, 128), (128, 2, B.KVQ_FP32, B.KVQ_META_FP8_BF16, 32), (64, 2, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 64)]


def _attend(fmt, rows, current, cached, q_scale=1.0, k_scale=1.0, v_scale=1.0, offset=None, spike=2.0, keys_and_values=None,
            poison=None):
    dim, bits, io, meta, group = fmt
    heads = 2
    dtype = torch.bfloat16 if io == B.KVQ_BF16 else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(4)

    def t(tokens, scale):
        return torch.randn((tokens, heads, dim), generator=gen, device=DEV) * scale

    cache = B.Cache(B.make_desc(heads, dim, bits, max(cached, 32), io, group, 1, meta), DEV)
    if cached:
        k, v = t(cached, k_scale), t(cached, v_scale)
        if offset:                    # every third token: all rotated channels far from 0, next to a small range
            for x in (k, v):
                x[::3] *= 1e-2 / offset
                x[::3, :, 0] += spike
        if keys_and_values:
            keys_and_values(k, v)
        B.kvq_quantize_append(cache, k.to(dtype), v.to(dtype))
    q = t(rows, q_scale).to(dtype)
    k, v = (t(current, k_scale).to(dtype), t(current, v_scale).to(dtype)) if current else (None, None)
    if poison:
        poison(q, k, v)
    got, mass = torch.full_like(q, float("nan")), torch.full((heads, rows), float("nan"), device=DEV)
    ref, ref_mass = torch.empty_like(got), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, cached, q, k, v, got, mass)
    B.kvq_chunk_attention_fp32(cache, 0, cached, q, k, v, ref, ref_mass)
    torch.cuda.synchronize()
    return cache, got, mass, ref, ref_mass


def _close(got, mass, ref, ref_mass, score_error=1e-5):
    """score_error: absolute error of a score, which weights, outputs and masses follow relatively; BF16 outputs may round the
    other way besides (2^-9 of the result)."""
    tol = score_error + (2.0 ** -9 if got.dtype == torch.bfloat16 else 0.0)
    assert torch.isfinite(ref).all() and torch.isfinite(got).all()
    assert float((got.double() - ref.double()).norm()) <= tol * float(ref.double().norm())
    torch.testing.assert_close(mass, ref_mass, rtol=10 * score_error, atol=1e-9)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("cached,current", [(32, 0), (0, 33), (7 * 32, 1), (8 * 32, 0), (5 * 32 + 3, 4 * 32), (9 * 32, 31), (40, 300), (20 * 32 + 1, 7 * 32 + 1)])
def test_runs_of_waves(fmt, cached, current):
    """Fewer tiles than waves, as many, one more; waves that go from cached to current tiles, and none that do."""
    _close(*_attend(fmt, 37, current, cached)[1:])


@pytest.mark.parametrize("fmt", FORMATS)
def test_zero_points_beyond_the_pieces(fmt):
    cache, *results = _attend(fmt, 40, 20, 300, offset=40.0)
    zero = B.export_all(cache, 0)[2].abs()
    assert (240.0 if fmt[3] == B.KVQ_META_FP32 else 15.0) < float(zero.max()) < 8192.0 and float(zero.min()) < 15.0
    # such a token's score and output are sums of terms zero / (2^bits - 1) times larger than their result: |zero| < 2^13,
    # 2^13 * 2^-24 relative to scores of a few units
    _close(*results, score_error=1e-3)


@pytest.mark.parametrize("fmt", [f for f in FORMATS if f[3] == B.KVQ_META_FP32])
@pytest.mark.parametrize("scales", [dict(q_scale=1e-32, k_scale=1e32), dict(q_scale=2.0 ** 105, k_scale=2.0 ** -105), dict(v_scale=1e-32),
                                    dict(v_scale=1e32)])
def test_ends_of_the_range(fmt, scales):
    # ordinary scores and weights throughout
    _close(*_attend(fmt, 40, 70, 200, **scales)[1:], score_error=2e-5)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("value", [math.inf, -math.inf, math.nan])
@pytest.mark.parametrize("where", ["q", "k", "v"])
def test_not_finite(fmt, value, where):
    def poison(q, k, v):
        {"q": q, "k": k, "v": v}[where][5, 0, 7] = value

    _, got, mass, ref, ref_mass = _attend(fmt, 40, 70, 200, poison=poison)
    for a, b in ((got, ref), (mass, ref_mass)):
        assert torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(torch.isposinf(a), torch.isposinf(b))
        ok = torch.isfinite(b)
        assert torch.equal(torch.isneginf(a), torch.isneginf(b)) and ok.any()
        torch.testing.assert_close(a[ok], b[ok], rtol=2.0 ** -7 if a.dtype == torch.bfloat16 else 1e-4, atol=1e-2 if a.dtype == torch.bfloat16 else 1e-5)


@pytest.mark.parametrize("fmt", [f for f in FORMATS if f[2] == B.KVQ_FP32])
def test_products_beyond_the_range(fmt):
    """A key whose score is -infinity in fp32 although query and key are ordinary numbers (1.1e21 .. and -1.7e21 in one channel)."""
    def poison(q, k, v):
        q[:, :, 7] = k[:, :, 7] = 0.0
        q[5:25, :, 7], k[3, :, 7] = 1.1e21 * 1.03 ** torch.arange(20, device=DEV)[:, None], -1.7e21

    _close(*_attend(fmt, 40, 70, 0, poison=poison)[1:])


# (E4M3 steps end at 448: no such cached values)
@pytest.mark.parametrize("large,fmt", [(large, f) for f in FORMATS for large in ("current", "cached", "both")
                                       if large == "current" or f[3] == B.KVQ_META_FP32])
def test_large_values_behind_a_late_maximum(fmt, large, monkeypatch):
    """Values of 2^119 at keys that score 7.5 (log2) above everything before them: what is summed stays within fp32 only where
    weights are taken relative to the largest score so far, whatever the reference was before."""
    dim, bits, io, meta, group = fmt
    monkeypatch.setattr(B, "_workspace", lambda *args: None)       # unsplit: a run of five tiles for each of the eight waves
    heads, rows, tokens, scale = 2, 33, 1280, 2.0 ** -3
    dtype = torch.bfloat16 if io == B.KVQ_BF16 else torch.float32
    # channel 1 rotates into alternating signs, which the codes hold exactly
    x = torch.zeros((tokens, heads, dim), device=DEV)
    x[..., 1] = 1e-3
    x[130::160, :, 1] = 7.5 * math.log(2.0) / scale
    v = torch.ones((tokens, heads, dim), device=DEV)
    v[:, :, 1::2] = -1.0
    v[130::160] *= 2.0 ** 119
    k, v = x.to(dtype), v.to(dtype)
    q = torch.zeros((rows, heads, dim), device=DEV)
    q[..., 1] = 1.0
    q = q.to(dtype)
    cache = B.Cache(B.make_desc(heads, dim, bits, tokens, io, group, 1, meta), DEV)
    cached = 0 if large == "current" else tokens
    if cached:
        B.kvq_quantize_append(cache, k, v)
    cur = (None, None) if large == "cached" else (k, v)
    got, mass = torch.full_like(q, float("nan")), torch.full((heads, rows), float("nan"), device=DEV)
    ref, ref_mass = torch.empty_like(got), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, cached, q, *cur, got, mass, scale, 0)
    B.kvq_chunk_attention_fp32(cache, 0, cached, q, *cur, ref, ref_mass, scale, 0)
    torch.cuda.synchronize()
    assert float(ref.abs().max()) > 2.0 ** 117
    _close(got.double() * 2.0 ** -119, mass, ref.double() * 2.0 ** -119, ref_mass, 1e-5 if io == B.KVQ_FP32 else 2.0 ** -8)


GROUPED = [(dim, bits, B.KVQ_FP32, B.KVQ_META_FP8_BF16, group) for dim in (64, 128) for bits in (2, 4) for group in (32, 64, 128) if group <= dim] + \
    [(64, 4, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 32), (64, 4, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 64)]


def _one_sided(k, v):
    """What ordinary data with one large channel and an offset of the values look like behind the rotation: groups of channels
    whose range does not hold 0, with zero-points of -30 .. 50 beside ordinary ones."""
    k[..., 32] *= 10.0
    v[..., 0] += 2.0 * math.sqrt(v.shape[2])
    v[: v.shape[0] // 2, :, 0] *= -1.0


@pytest.mark.parametrize("fmt", GROUPED)
@pytest.mark.parametrize("large", ["keys", "values", "both"])
def test_groups_whose_range_does_not_hold_zero(fmt, large):
    def change(k, v):
        a, b = k.clone(), v.clone()
        _one_sided(a, b)
        if large != "values":
            k.copy_(a)
        if large != "keys":
            v.copy_(b)

    cache, *results = _attend(fmt, 40, 70, 300, q_scale=0.3, keys_and_values=change)
    low, high = (-12.0, 15.0) if fmt[1] == 2 else (0.0, 15.0)
    if fmt[1] == 4 and (large == "values" or fmt[4] == 32):      # beyond what one operand holds, next to ordinary ones
        zero = B.export_all(cache, 0 if large == "keys" else 1)[2]
        out = (zero < low) | (zero > high)
        assert 0.005 < float(out.float().mean()) and float(zero.abs().max()) < 128.0
    # a score or an output is a sum of terms |zero| / 15 < 8 times larger than without the offset
    _close(*results, score_error=8e-5)


@pytest.mark.parametrize("fmt", GROUPED)
def test_zero_points_beyond_exact_constants(fmt):
    """Zero-points above 2^20: fp32 products, where the scores are as inexact as fp32 makes them."""
    cache, *results = _attend(fmt, 40, 70, 200, q_scale=1e-5, offset=4e4, spike=4200.0 * math.sqrt(fmt[0]))
    assert float(B.export_all(cache, 0)[2].abs().max()) > 2.0 ** 20
    # |q~| * zero * step * 2^-24 = 1e-5 * 4200 * sqrt(dim) * 2^-24 in a score
    _close(*results, score_error=1e-5)


@pytest.mark.parametrize("fmt", [(64, 4, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 32), (128, 4, B.KVQ_FP32, B.KVQ_META_FP8_BF16, 32)])
def test_such_groups_take_about_the_usual_time(fmt):
    dim, bits, io, meta, group = fmt
    heads, rows, cached = 8, 256, 2000
    dtype = torch.bfloat16 if io == B.KVQ_BF16 else torch.float32
    calls = []
    for one_sided in (False, True):
        k, v = (torch.randn((cached, heads, dim), device=DEV) for _ in range(2))
        if one_sided:
            _one_sided(k, v)
        cache = B.Cache(B.make_desc(heads, dim, bits, cached, io, group, 1, meta), DEV)
        B.kvq_quantize_append(cache, k.to(dtype), v.to(dtype))
        q = torch.randn((rows, heads, dim), device=DEV).to(dtype)
        out = torch.empty_like(q)
        calls.append(lambda cache=cache, q=q, out=out: B.kvq_chunk_attention(cache, 0, cached, q, None, None, out))
    times = [math.inf, math.inf]
    for _ in range(5):
        for i, call in enumerate(calls):
            call()
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(50):
                call()
            end.record()
            end.synchronize()
            times[i] = min(times[i], begin.elapsed_time(end))
    # 2.3 to 2.6 times as long while such tiles took the fp32 matrix instructions
    assert times[1] < 1.6 * times[0], times
