"""The 2-bit matrix-core kernel's query pieces (rotated on the matrix cores, four FP6 pieces per row), with keys per token and per
channel, against the vector kernel: key blocks of one token, shorter than a tile, ending inside one, of whole tiles; row counts
around the 32 and 64 rows of a wave; channel signs; one key channel that dwarfs the others."""
import math

import pytest
import torch

from launches import SIXTEEN_BIT, attention_threads
from paper_2605_26266_amd import binding as B
from test_gpu_attention import P                                                                                  # noqa: F401

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("rows,signs,outlier", [(1, False, 0.0), (31, True, 0.0), (33, False, 4.0), (65, True, 4.0), (257, False, 0.0)])
@pytest.mark.parametrize("blocks", [(1,), (32,), (37, 1), (200, 37, 96, 1), (256, 256)])
@pytest.mark.parametrize("axis,correction", [(B.KVQ_KEYS_PER_CHANNEL, 0), (B.KVQ_KEYS_PER_CHANNEL, 1), (B.KVQ_KEYS_PER_TOKEN, 0), (B.KVQ_KEYS_PER_TOKEN, 1)])
def test_query_pieces(P, axis, correction, blocks, rows, signs, outlier):        # noqa: F811
    heads, current = 2, 40
    if axis == B.KVQ_KEYS_PER_TOKEN:
        rows += 12288          # (the fp32 kernel takes fewer; three rounds of its 256 workgroups, one of the 16-bit kernel's)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(21)

    def t(n, shift=0.0):       # the shift is one rotated channel
        x = torch.randn((n, heads, 128), generator=gen, device=DEV)
        return (x + shift * torch.randn((n, heads, 1), generator=gen, device=DEV)).to(torch.bfloat16)

    cache = B.Cache(B.make_desc(heads, 128, 2, -(-sum(blocks) // 32) * 32 + 32, B.KVQ_BF16, key_axis=axis), DEV)
    if signs:
        B.kvq_cache_set_rotation_signs(cache, [(5 * i * i + i) % 7 < 3 for i in range(128)])
    for n in blocks:
        B.kvq_quantize_append(cache, t(n, outlier), t(n))
    q, k, v = t(rows), t(current), t(current)
    out, mass = torch.full_like(q, float("nan")), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, sum(blocks), q, k, v, out, mass, correction=correction)
    B.kvq_chunk_attention_fp32(cache, 0, sum(blocks), q, k, v, ref, ref_mass, correction=correction)
    ws = B._workspace(cache, 0, sum(blocks), rows, current, 1, None)
    assert attention_threads(cache, 0, sum(blocks), q, k, v, out, correction=correction, workspace=ws) == SIXTEEN_BIT
    torch.cuda.synchronize()
    # 2^e0 < max / 3.75 and the pieces leave at most 2^(e0 - 15) of every channel, which meets a code of at most 3: a score is off
    # by no more than 3 * 128 * 2^-15 / 3.75 = 2^-8.3 of the row's largest |rotated query * step| * sigma.  The query's norm,
    # sqrt(128 + log terms) < 16, bounds a rotated channel.  The row constants are bf16 pieces (2^-24 of them) and sums fp32.
    steps = B.export_all(cache, 0)[1]
    score_error = 2.0 ** -8.3 * 16.0 * float(steps.max()) / math.sqrt(128.0)
    # The bar is one against exact outputs; these are rounded to BF16 too, by at most 2^-8 of themselves.
    bar = P.TOL_OUT_BF16 + 2.0 ** -8 * float(ref.abs().max())
    # (below 1e-3 the fp32 format of P_S, 6e-8 near 1, would take a share of the relative bar on 1 - P_S)
    P.assert_attention_close(out.double().cpu().numpy(), mass.double().cpu().numpy(), ref.double().cpu().numpy(),
                             ref_mass.double().cpu().numpy(), bar, "query pieces", mass_floor=1e-3)
    assert float((mass.double() / ref_mass.double()).log().abs().max()) <= score_error


@pytest.mark.parametrize("axis", [B.KVQ_KEYS_PER_TOKEN, B.KVQ_KEYS_PER_CHANNEL])
def test_norms_of_large_queries(P, axis):        # noqa: F811
    """Queries of norm 8e18, whose square is within fp32 and 128 times the square is not; ordinary scores and corrections."""
    heads, rows, cached, current, scale = 4, 3000, 200, 40, 1.2e-19
    gen = torch.Generator(device=DEV)
    gen.manual_seed(9)

    def t(n, times=1.0):
        return (torch.randn((n, heads, 128), generator=gen, device=DEV) * times).to(torch.bfloat16)

    cache = B.Cache(B.make_desc(heads, 128, 2, 224, B.KVQ_BF16, key_axis=axis), DEV)
    B.kvq_quantize_append(cache, t(cached), t(cached))
    q, k, v = t(rows, 7e17), t(current), t(current)
    out, mass = torch.full_like(q, float("nan")), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, cached, q, k, v, out, mass, scale)
    B.kvq_chunk_attention_fp32(cache, 0, cached, q, k, v, ref, ref_mass, scale)
    torch.cuda.synchronize()
    assert attention_threads(cache, 0, cached, q, k, v, out) == SIXTEEN_BIT
    P.assert_attention_close(out.double().cpu().numpy(), mass.double().cpu().numpy(), ref.double().cpu().numpy(),
                             ref_mass.double().cpu().numpy(), P.TOL_OUT_BF16, "large queries")
