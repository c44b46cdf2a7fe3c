"""The fp32 matrix-core attention kernel (per-token caches outside BF16 / head_dim 128) against the vector kernel, which
computes the same expressions in fp32 in another order."""
import pytest
import torch

from paper_2605_26266_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (dim, bits, io, meta, group)
FORMATS = [(64, 2, B.KVQ_FP32, B.KVQ_META_FP32, 64), (64, 4, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 32),
           (64, 2, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 64), (128, 2, B.KVQ_FP32, B.KVQ_META_FP32, 128),
           (128, 4, B.KVQ_FP32, B.KVQ_META_FP8_BF16, 32), (128, 2, B.KVQ_FP32, B.KVQ_META_FP8_BF16, 64),
           (128, 4, B.KVQ_FP32, B.KVQ_META_FP8_BF16, 128)]
# (heads, ratio, rows, current keys, causal, slid past, appended blocks, first cached token, cached tokens, signs)
SHAPES = [
    (1, 1, 1, 0, False, 0, [1], 0, 1, False),
    (2, 1, 33, 31, False, 0, [64], 0, 64, False),
    (3, 2, 40, 45, True, 17, [100, 61], 5, 140, True),       # ragged window in a ring, rows that see part of a tile
    (1, 4, 7, 300, True, 0, [], 0, 0, False),                # no cached tokens; split: early rows see no key of late pieces
    (2, 1, 70, 64, False, 0, [3000], 1, 2998, False),        # split over workgroups
    (300, 1, 5, 3, False, 0, [40], 0, 40, False),            # more units than compute units
]


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("shape", SHAPES)
def test_agrees_with_the_vector_kernel(fmt, shape):
    dim, bits, io, meta, group = fmt
    heads, ratio, rows, current, causal, slid, blocks, start, length, signs = shape
    dtype = torch.bfloat16 if io == B.KVQ_BF16 else torch.float32
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)

    def t(tokens, h):
        return torch.randn((tokens, h, dim), generator=gen, device=DEV).to(torch.bfloat16).to(dtype)

    cache = B.Cache(B.make_desc(heads, dim, bits, max(sum(blocks), 32) + 32, io, group, 1, meta), DEV)
    if signs:
        B.kvq_cache_set_rotation_signs(cache, [(7 * c) % 5 < 2 for c in range(dim)])
    if slid:
        B.kvq_quantize_append(cache, t(slid, heads), t(slid, heads))
    for i, n in enumerate(blocks):
        B.kvq_quantize_append(cache, t(n, heads), t(n, heads))
        if i == 0 and slid:
            B.kvq_cache_evict(cache, slid)
    q = t(rows, heads * ratio)
    k, v = (t(current, heads), t(current, heads)) if current else (None, None)
    out = torch.full_like(q, float("nan"))
    mass = torch.full((heads * ratio, rows), float("nan"), dtype=torch.float32, device=DEV)
    B.kvq_chunk_attention_ex(cache, start, length, q, k, v, out, mass, causal=causal)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    for j in range(ratio):
        for r in (range(rows) if causal else [slice(0, rows)]):
            rs = slice(r, r + 1) if causal else r
            seen = current - rows + r + 1 if causal else current
            qj = torch.empty((q[rs].shape[0], heads, dim), dtype=dtype, device=DEV).copy_(q[rs, j::ratio])
            o, p = torch.empty_like(qj), torch.empty((heads, qj.shape[0]), dtype=torch.float32, device=DEV)
            B.kvq_chunk_attention_fp32(cache, start, length, qj, k[:seen] if current else None, v[:seen] if current else None, o, p)
            ref[rs, j::ratio] = o
            ref_mass[j::ratio, rs] = p
    torch.cuda.synchronize()
    # A score is a sum of dim + 1 products with |s| below about 2^6 after softmax relevance: dim * 2^-24 * 2^6 / sqrt(dim) < 5e-5
    # absolute in the exponent at worst, 1e-6 for typical sums; weights, outputs and masses follow it relatively.
    rel = float((out.double() - ref.double()).norm() / ref.double().norm())
    assert rel <= (1e-5 if dtype == torch.float32 else 2.0 ** -9)      # BF16 outputs: ties rounded the other way
    assert float((out.double() - ref.double()).abs().max()) <= (1e-4 if dtype == torch.float32 else 2.0 ** -7 * float(ref.abs().max()))
    torch.testing.assert_close(mass, ref_mass, rtol=5e-5, atol=1e-9)


def test_what_the_window_leaves_out_does_not_reach_the_result():
    """Non-finite tokens beside the window, in its first and last tile, and beside the current block."""
    cache = B.Cache(B.make_desc(2, 64, 2, 160, B.KVQ_FP32), DEV)
    x = torch.randn((96, 2, 64), device=DEV)
    x[:5] = float("inf")
    x[90:] = float("nan")
    B.kvq_quantize_append(cache, x, x)
    k = torch.randn((40, 2, 64), device=DEV)
    out, mass = torch.empty((9, 2, 64), device=DEV), torch.empty((2, 9), device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    q = torch.randn((9, 2, 64), device=DEV)
    B.kvq_chunk_attention(cache, 5, 85, q, k, k, out, mass)
    B.kvq_chunk_attention_fp32(cache, 5, 85, q, k, k, ref, ref_mass)
    assert torch.isfinite(out).all() and torch.isfinite(ref).all()
    torch.testing.assert_close(out, ref, rtol=1e-4, atol=1e-5)
    torch.testing.assert_close(mass, ref_mass, rtol=5e-5, atol=1e-9)


@pytest.mark.parametrize("correction", [0, 1])
@pytest.mark.parametrize("dim,bits", [(64, 2), (128, 4)])
def test_steps_whose_square_overflows(dim, bits, correction):
    """Keys of about 1e19 .. 1e20 against queries as small: the scores and the correction are ordinary numbers."""
    heads, tokens, rows = 2, 150, 40
    gen = torch.Generator(device=DEV)
    gen.manual_seed(2)
    k = torch.randn((tokens, heads, dim), generator=gen, device=DEV)
    k *= 10.0 ** (18.5 + 1.5 * torch.rand((tokens, 1, 1), generator=gen, device=DEV))      # steps on either side of 2^64
    v, cur = (torch.randn((n, heads, dim), generator=gen, device=DEV) for n in (tokens, 20))
    q = torch.randn((rows, heads, dim), generator=gen, device=DEV) * 4e-20
    cache = B.Cache(B.make_desc(heads, dim, bits, 160, B.KVQ_FP32), DEV)
    B.kvq_quantize_append(cache, k, v)
    step = B.export_all(cache, 0)[1]
    assert 0 < int((step >= 2.0 ** 64).sum()) < step.numel()
    out, mass = torch.empty_like(q), torch.empty((heads, rows), device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass, correction=correction)
    B.kvq_chunk_attention_fp32(cache, 0, tokens, q, cur, cur, ref, ref_mass, correction=correction)
    assert torch.isfinite(ref).all() and torch.isfinite(out).all()
    # |q|^2 sigma^2 / 24 is about 1e-41 here, 2^13 steps of the denormal grid: the correction (below 1) is good to 2^-13
    torch.testing.assert_close(out, ref, rtol=1e-3, atol=1e-3)
    torch.testing.assert_close(mass, ref_mass, rtol=1e-3, atol=1e-6)
