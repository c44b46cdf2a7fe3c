"""The oracle tests of the attention calls once more on the 16-bit matrix kernels.  Calls over a few query rows or keys of the caches
that these kernels serve are estimated to be faster on the fp32 kernel, which takes the tests' shapes; here the same query rows come
behind thousands of copies of themselves, every call is checked to launch a 16-bit kernel, and the copies are compared too."""
import numpy as np
import pytest
import torch

from launches import FP32, SIXTEEN_BIT, attention_threads
from paper_2605_26266_amd import binding as B
from test_gpu_attention import (P, test_all_zero_vectors_in_the_cache, test_extreme_key_and_value_scales,             # noqa: F401
                                test_group_wise_fp8_metadata, test_large_zero_points, test_large_zero_points_fp8_bf16_metadata,
                                test_query_dynamic_range, test_ragged_shapes_and_windows, test_randomised_rotation_signs,
                                test_ring_of_two_tiles, test_seeded_sweep_of_rings_and_windows, test_sliding_window_ring,
                                test_small_all_rows, test_softmax_scale_and_large_queries, test_zero_points_beyond_the_matrix_core_domain)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ROWS = 3 * 256 * 32      # rows over all heads that take the fp32 kernel three rounds of 256 workgroups, the 16-bit kernels one


def _long_call(cache, q, k_cur, v_cur, io_dtype, cache_start=0, cache_len=None, correction=1, softmax_scale=0.0):
    import parity
    length = len(cache) - cache_start if cache_len is None else cache_len
    rows, heads = q.shape[:2]
    pad = -(-ROWS // (heads * 256)) * 256          # the rows themselves lie in their blocks as they would alone
    source = (np.arange(pad + rows) - pad) % rows
    qd = parity.to_dev(q, io_dtype)[torch.from_numpy(source).to(DEV)].contiguous()
    kd, vd = (parity.to_dev(x, io_dtype) if x is not None and x.shape[0] else None for x in (k_cur, v_cur))
    out = torch.full_like(qd, float("nan"))
    mass = torch.full((heads, pad + rows), float("nan"), dtype=torch.float32, device=DEV)
    B.kvq_chunk_attention(cache, cache_start, length, qd, kd, vd, out, mass, softmax_scale, correction)
    ws = B._workspace(cache, cache_start, length, pad + rows, 0 if kd is None else kd.shape[0], 1, None)
    assert attention_threads(cache, cache_start, length, qd, kd, vd, out, correction=correction, workspace=ws) == SIXTEEN_BIT
    torch.cuda.synchronize()
    out, mass = out.float().cpu().numpy().astype(np.float64), mass.cpu().numpy().astype(np.float64)
    last, last_mass = out[pad:], mass[:, pad:]
    assert np.max(np.abs(out - last[source])) <= parity.TOL_OUT_BF16 * max(1.0, np.max(np.abs(last)))
    # (a row's reference follows the rows beside it: the copies differ in rounding)
    assert np.all(np.abs(mass - last_mass[:, source]) <= 2 * parity.TOL_MASS_REL * last_mass[:, source] + parity.MASS_FLOOR)
    return last, last_mass


@pytest.fixture(autouse=True, params=[True, False], ids=["split", "unsplit"])
def long_calls(request, monkeypatch):
    import parity
    short = parity.run_gpu_attention

    def run(*args, fp32_kernel=False, causal=None, **kw):
        if fp32_kernel or args[4] == "fp32":
            return short(*args, fp32_kernel=fp32_kernel, causal=causal, **kw)
        assert causal is None
        return _long_call(*args, **kw)

    monkeypatch.setattr(parity, "run_gpu_attention", run)
    if not request.param:
        monkeypatch.setattr(B, "_workspace", lambda *args: None)


@pytest.mark.parametrize("bits,group", [(2, 128), (4, 128), (2, 32), (2, 64), (4, 32), (4, 64)])
@pytest.mark.parametrize("cached", [500, 0])
def test_grouped_heads_and_a_causal_block(P, bits, group, cached):        # noqa: F811
    """Six query heads over two key/value heads, causal current block: one long call against calls over 100 of its rows each, which
    end with the last key that those rows see and run on the fp32 kernel."""
    heads, ratio, rows, current = 2, 3, 4096, 4099
    gen = torch.Generator(device=DEV)
    gen.manual_seed(17)

    def t(n, h):
        return torch.randn((n, h, 128), generator=gen, device=DEV).to(torch.bfloat16)

    meta = B.KVQ_META_FP32 if group == 128 else B.KVQ_META_FP8_BF16
    cache = B.Cache(B.make_desc(heads, 128, bits, max(cached, 32), B.KVQ_BF16, group, 1, meta), DEV)
    if cached:
        B.kvq_quantize_append(cache, t(cached, heads), t(cached, heads))
    q, k, v = t(rows, heads * ratio), t(current, heads), t(current, heads)
    out, mass = torch.full_like(q, float("nan")), torch.empty((heads * ratio, rows), dtype=torch.float32, device=DEV)
    B.kvq_chunk_attention_ex(cache, 0, cached, q, k, v, out, mass, causal=True)
    ws = B._workspace(cache, 0, cached, rows, current, ratio, None)
    assert attention_threads(cache, 0, cached, q, k, v, out, causal=True, workspace=ws) == SIXTEEN_BIT
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    for r in range(0, rows, 100):
        r1 = min(r + 100, rows)
        seen = current - rows + r1
        part, part_mass = torch.empty_like(q[r:r1]), torch.empty((heads * ratio, r1 - r), dtype=torch.float32, device=DEV)
        args = cache, 0, cached, q[r:r1], k[:seen], v[:seen], part
        B.kvq_chunk_attention_ex(*args, part_mass, causal=True)
        if r == 0:
            ws = B._workspace(cache, 0, cached, r1, seen, ratio, None)
            assert attention_threads(*args, causal=True, workspace=ws) == FP32
        ref[r:r1], ref_mass[:, r:r1] = part, part_mass
    torch.cuda.synchronize()
    P.assert_attention_close(out.double().cpu().numpy(), mass.double().cpu().numpy(), ref.double().cpu().numpy(),
                             ref_mass.double().cpu().numpy(), P.TOL_OUT_BF16, "causal", mass_floor=1e-4)


@pytest.mark.parametrize("bits,group,axis", [(2, 128, 0), (4, 128, 0), (2, 32, 0), (4, 32, 0), (4, 64, 0), (2, 128, 1), (4, 128, 1)])
def test_flagged_cache_is_served_by_the_vector_kernel(bits, group, axis):
    """The launch of the 16-bit kernel leaves a flagged cache to the one behind it, whose results are the vector kernel's bit for bit."""
    heads, tokens, rows = 3, 300, ROWS // 3 + 70
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    fp8 = group != 128
    k = torch.randn((tokens, heads, 128), generator=gen, device=DEV) * (1e-3 if fp8 else 1e-5)
    k[..., 0] += 4000.0 if fp8 else 40.0               # E4M3 steps are at least 2^-9
    v, q, cur = (torch.randn((n, heads, 128), generator=gen, device=DEV).to(torch.bfloat16) for n in (tokens, rows, 64))
    q *= 2e-4 if fp8 else 0.02
    cache = B.Cache(B.make_desc(heads, 128, bits, tokens, B.KVQ_BF16, group, 1, B.KVQ_META_FP8_BF16 if fp8 else B.KVQ_META_FP32, axis), DEV)
    B.kvq_quantize_append(cache, k.to(torch.bfloat16), v)
    assert float(B.export_all(cache, 0)[2].abs().max()) > 65536.0
    out, mass = torch.full_like(q, float("nan")), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass)
    B.kvq_chunk_attention_fp32(cache, 0, tokens, q, cur, cur, ref, ref_mass)
    ws = B._workspace(cache, 0, tokens, rows, 64, 1, None)
    assert attention_threads(cache, 0, tokens, q, cur, cur, out, workspace=ws) == SIXTEEN_BIT
    torch.cuda.synchronize()
    assert torch.isfinite(ref).all() and torch.equal(out, ref) and torch.equal(mass, ref_mass)
