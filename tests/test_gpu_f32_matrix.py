"""The fp32 matrix-core attention kernel (per-token caches outside BF16 / head_dim 128, and calls of those caches over a few
query rows) against the vector kernel, which computes the same expressions in fp32 in another order."""
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
    (1, 4, 7, 300, True, 0, [], 0, 0, False),                # no cached tokens
    (2, 1, 70, 64, False, 0, [3000], 1, 2998, False),        # split over workgroups
    (300, 1, 5, 3, False, 0, [40], 0, 40, False),            # more units than compute units
]
# the same; all split
SPLIT_SHAPES = [
    (2, 1, 900, 900, True, 0, [], 0, 0, False),              # pieces without a key that the rows of the block see
    (300, 1, 5, 3, False, 0, [1000], 0, 1000, False),        # 256 whole units and 44 in pieces
]
# BF16, head_dim 128: (bits, meta, group), one shape per kind of call that a few rows take to this kernel
FEW_ROW_FORMATS = [(b, B.KVQ_META_FP32, 128) for b in (2, 4)] + [(b, B.KVQ_META_FP8_BF16, g) for b in (2, 4) for g in (32, 64, 128)]
FEW_ROW_SHAPES = [
    (8, 4, 1, 64, False, 0, [8192], 0, 8192, False),         # a row per query head, four heads in a unit
    (8, 4, 3, 41, True, 17, [3000, 3100], 5, 6090, True),    # ragged window in a ring, rows that see part of a tile
    (260, 2, 3, 5, True, 0, [1000], 0, 1000, False),         # 256 whole units and 4 in pieces
]


def _pieces(cache, start, length, rows, current, ratio):
    """Pieces of 32 rows that the call's work space has room for (every unit of the fp32 kernel is one block of 32 rows)."""
    nbytes = B.lib().kvq_attention_workspace_bytes(cache.handle, start, length, rows, current, ratio)
    return nbytes // (32 * (cache.desc.head_dim + 4) * 4)


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("shape", SHAPES + SPLIT_SHAPES)
def test_agrees_with_the_vector_kernel(fmt, shape):
    cache, q, k, v, out, mass = _run(fmt, shape)
    if shape in SPLIT_SHAPES:
        assert _pieces(cache, shape[7], shape[8], shape[2], shape[3], shape[1]) > 0
    _compare(cache, shape, q, k, v, out, mass)


@pytest.mark.parametrize("fmt", FEW_ROW_FORMATS)
@pytest.mark.parametrize("shape", FEW_ROW_SHAPES)
def test_few_rows_of_caches_of_the_16_bit_kernels(fmt, shape):
    heads, ratio = shape[:2]
    cache, q, k, v, out, mass = _run((128, fmt[0], B.KVQ_BF16, *fmt[1:]), shape)
    # The 16-bit kernels would have a unit per query head, this one has a unit per key/value head: the pieces are a multiple of
    # the units left over from whole rounds of 256 workgroups.
    pieces = _pieces(cache, shape[7], shape[8], shape[2], shape[3], ratio)
    assert pieces > 0 and pieces % (heads % 256) == 0 and pieces % (heads * ratio % 256) != 0, "meant for the fp32 kernel"
    _compare(cache, shape, q, k, v, out, mass)


@pytest.mark.parametrize("fmt", [FORMATS[0], FORMATS[1], (128, 2, B.KVQ_BF16, B.KVQ_META_FP8_BF16, 64)])
@pytest.mark.parametrize("option", ["strides", "uncorrected", "stream"])
def test_options(fmt, option):
    shape = (8, 4, 3, 41, True, 17, [1000, 1100], 5, 2090, True)
    cache, q, k, v, out, mass = _run(fmt, shape, option)
    _compare(cache, shape, q, k, v, out, mass, int(option != "uncorrected"))


def test_flagged_cache_over_few_rows():
    """Zero-points beyond the 16-bit kernels' domain are no matter here: no other kernel steps in."""
    heads, ratio, tokens = 8, 4, 8192
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    k = torch.randn((tokens, heads, 128), generator=gen, device=DEV) * 1e-5
    k[..., 0] += 40.0
    v = torch.randn((tokens, heads, 128), generator=gen, device=DEV).to(torch.bfloat16)
    cache = B.Cache(B.make_desc(heads, 128, 2, tokens, B.KVQ_BF16), DEV)
    B.kvq_quantize_append(cache, k.to(torch.bfloat16), v)
    assert float(B.export_all(cache, 0, 0, 1)[2].abs().max()) > 65500.0
    pieces = _pieces(cache, 0, tokens, 1, 64, ratio)
    assert pieces > 0 and pieces % (heads * ratio) != 0, "meant for the fp32 kernel"
    q = (torch.randn((1, heads * ratio, 128), generator=gen, device=DEV) * 0.02).to(torch.bfloat16)
    cur = torch.randn((64, heads, 128), generator=gen, device=DEV).to(torch.bfloat16)
    out, mass = torch.empty_like(q), torch.empty((heads * ratio, 1), dtype=torch.float32, device=DEV)
    B.kvq_chunk_attention_ex(cache, 0, tokens, q, cur, cur, out, mass)
    _compare(cache, (heads, ratio, 1, 64, False, 0, [], 0, tokens, False), q, cur, cur, out, mass)


def _run(fmt, shape, option=None):
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
    if option == "strides":       # every second head and the first channels of wider tensors
        q, k, v, out = (torch.cat([x, x.flip(0)], 2).repeat_interleave(2, 1)[:, ::2, :dim] for x in (q, k, v, out))
        assert not q.is_contiguous() and q.stride(1) == 4 * dim
    mass = torch.full((heads * ratio, rows), float("nan"), dtype=torch.float32, device=DEV)
    if option == "stream":
        stream = torch.cuda.Stream()
        stream.wait_stream(torch.cuda.current_stream())
        B.kvq_chunk_attention_ex(cache, start, length, q, k, v, out, mass, causal=causal, stream=stream)
        torch.cuda.current_stream().wait_stream(stream)
    else:
        B.kvq_chunk_attention_ex(cache, start, length, q, k, v, out, mass, causal=causal, correction=int(option != "uncorrected"))
    return cache, q, k, v, out, mass


def _compare(cache, shape, q, k, v, out, mass, correction=1):
    heads, ratio, rows, current, causal, _, _, start, length, _ = shape
    dim, dtype = cache.desc.head_dim, q.dtype
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    k, v = (None, None) if k is None else (k.contiguous(), v.contiguous())
    for j in range(ratio):
        for r in (range(rows) if causal else [slice(0, rows)]):
            rs = slice(r, r + 1) if causal else r
            seen = current - rows + r + 1 if causal else current
            qj = torch.empty((q[rs].shape[0], heads, dim), dtype=dtype, device=DEV).copy_(q[rs, j::ratio])
            o, p = torch.empty_like(qj), torch.empty((heads, qj.shape[0]), dtype=torch.float32, device=DEV)
            B.kvq_chunk_attention_fp32(cache, start, length, qj, k[:seen] if current else None, v[:seen] if current else None, o, p,
                                       correction=correction)
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
