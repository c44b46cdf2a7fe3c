"""The oracle tests of the attention calls once more without a work space: kvq_chunk_attention and kvq_chunk_attention_ex
themselves, nothing split.  And windows of a few tiles in the group-wise 16-bit kernels, which serve them where there are many
query rows (calls over few rows and tiles are estimated to be faster on the fp32 kernel)."""
import pytest
import torch

from paper_2605_26266_amd import binding as B
from test_gpu_attention import (P, test_group_wise_fp8_metadata, test_grouped_query_heads_and_causal_block,        # noqa: F401
                                test_ragged_shapes_and_windows, test_ring_of_two_tiles, test_seeded_sweep_of_rings_and_windows,
                                test_sliding_window_ring, test_small_all_rows, test_zero_points_beyond_the_matrix_core_domain)
from test_gpu_per_channel import (test_per_channel_keys, test_per_channel_keys_many_tiles,                       # noqa: F401
                                  test_per_channel_partly_evicted_block_and_grouped_heads, test_per_channel_ring_and_block_limit)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(autouse=True)
def no_workspace(monkeypatch):
    monkeypatch.setattr(B, "_workspace", lambda *args: None)


# (slid past, appended, first cached token, cached tokens): 3, 4, 6 and 8 tiles, at the end of the ring, round it, inside tiles
@pytest.mark.parametrize("window", [(0, 96, 0, 96), (64, 128, 0, 128), (70, 186, 7, 170), (17, 250, 1, 240)])
@pytest.mark.parametrize("bits,group", [(2, 32), (2, 64), (4, 32), (4, 64)])
def test_short_windows_of_the_group_wise_kernels(P, bits, group, window):        # noqa: F811
    slid, appended, start, length = window
    heads, rows, current = 4, 3000, 40
    gen = torch.Generator(device=DEV)
    gen.manual_seed(13)

    def t(n):
        return torch.randn((n, heads, 128), generator=gen, device=DEV).to(torch.bfloat16)

    cache = B.Cache(B.make_desc(heads, 128, bits, -(-appended // 32) * 32 + 32, B.KVQ_BF16, group, 1, B.KVQ_META_FP8_BF16), DEV)
    if slid:
        B.kvq_quantize_append(cache, t(slid), t(slid))
        B.kvq_cache_evict(cache, slid)
    B.kvq_quantize_append(cache, t(appended), t(appended))
    q, k, v = t(rows), t(current), t(current)
    out, mass = torch.full_like(q, float("nan")), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, start, length, q, k, v, out, mass)
    B.kvq_chunk_attention_fp32(cache, start, length, q, k, v, ref, ref_mass)
    torch.cuda.synchronize()
    # not the fp32 kernel: its masses agree with the vector kernel's to fp32 rounding, these sum f16-rounded weights (2^-11 each)
    assert float((mass / ref_mass - 1).abs().max()) > 1e-5
    P.assert_attention_close(out.double().cpu().numpy(), mass.double().cpu().numpy(), ref.double().cpu().numpy(),
                             ref_mass.double().cpu().numpy(), P.TOL_OUT_BF16, "short window")
