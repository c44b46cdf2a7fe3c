"""Calls whose key range is split over workgroups (kvq_chunk_attention_ws) against the same call unsplit."""
import ctypes

import pytest
import torch

from launches import SIXTEEN_BIT, attention_threads
from paper_2605_26266_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _call(cache, start, length, q, k, v, ratio, causal, workspace):
    """The C entry itself; workspace None: nothing is split."""
    out = torch.full_like(q, float("nan"))
    mass = torch.full((q.shape[1], q.shape[0]), float("nan"), dtype=torch.float32, device=DEV)
    n_cur = 0 if k is None else k.shape[0]
    opts = B.kvq_attention_opts(ratio, int(causal), q.stride(0), q.stride(1))
    heads, dim = cache.desc.num_heads, cache.desc.head_dim
    status = B.lib().kvq_chunk_attention_ws(
        cache.handle, start, length, q.data_ptr(), None if k is None else k.data_ptr(), None if v is None else v.data_ptr(),
        q.shape[0], n_cur, heads * dim, dim, 0.0, 1, ctypes.byref(opts), out.data_ptr(), mass.data_ptr(),
        None if workspace is None else workspace.data_ptr(), 0 if workspace is None else workspace.numel(),
        int(torch.cuda.current_stream().cuda_stream))
    assert status == B.KVQ_OK
    torch.cuda.synchronize()
    return out.float(), mass


FORMATS = [(2, B.KVQ_META_FP32, 128, 0), (4, B.KVQ_META_FP32, 128, 0), (2, B.KVQ_META_FP8_BF16, 32, 0),
           (4, B.KVQ_META_FP8_BF16, 64, 0), (2, B.KVQ_META_FP32, 128, 1)]
# (heads, ratio, rows, current keys, causal, appended blocks, first cached token, cached tokens)
SHAPES = [
    (1, 1, 1, 1, True, [2000], 0, 2000),              # one row, one current key
    (2, 3, 33, 70, True, [500, 269], 45, 700),       # ragged window over two blocks, rows that see part of a piece only
    (2, 4, 3, 40, True, [700, 50], 3, 747),          # few rows, grouped query heads
    (3, 1, 300, 1000, True, [96], 0, 96),            # pieces that hold current tiles alone, some invisible to early rows
    (8, 1, 257, 1, False, [1024], 31, 993),          # a second row block with one row
    (5, 1, 64, 0, False, [2000], 1, 1999),           # no current block
    (2, 1, 600, 857, False, [], 0, 0),               # no cached tokens
    (8, 1, 900, 1000, True, [3000], 5, 2990),        # 32 blocks of 256 rows in the 16-bit kernels
    (44, 1, 1600, 33, False, [2000], 0, 2000),       # 308 blocks: 256 whole, 52 split
]
# Keys per token: the last two above, and what the first ones stand for over rows enough for the 16-bit kernels
SIXTEEN_BIT_SHAPES = SHAPES[-2:] + [
    (2, 3, 2600, 2700, True, [500, 269], 45, 700),   # ragged window over two blocks, rows that see part of a piece only
    (3, 1, 6000, 6000, True, [96], 0, 96),           # pieces that hold current tiles alone, some invisible to early rows
    (8, 1, 1281, 1, False, [3024], 31, 2993),        # a last row block with one row
    (5, 1, 2100, 0, False, [4000], 1, 3999),         # no current block
    (2, 1, 8200, 8200, False, [], 0, 0),             # no cached tokens
]


@pytest.mark.parametrize("fmt", FORMATS)
@pytest.mark.parametrize("shape", SHAPES + SIXTEEN_BIT_SHAPES[2:])
def test_split_call_agrees_with_the_unsplit_one(fmt, shape):
    bits, meta, group, axis = fmt
    heads, ratio, rows, current, causal, blocks, start, length = shape
    gen = torch.Generator(device=DEV)
    gen.manual_seed(7)

    def t(tokens, h):
        return torch.randn((tokens, h, 128), generator=gen, device=DEV).to(torch.bfloat16)

    cache = B.Cache(B.make_desc(heads, 128, bits, max(sum(blocks), 32) + 64, B.KVQ_BF16, group, 1, meta, axis), DEV)
    for n in blocks:
        B.kvq_quantize_append(cache, t(n, heads), t(n, heads))
    q = t(rows, heads * ratio)
    k, v = (t(current, heads), t(current, heads)) if current else (None, None)
    largest = 6.0              # of the N(0, 1) values
    nbytes = B.lib().kvq_attention_workspace_bytes(cache.handle, start, length, rows, current, ratio)
    if axis == 0 or length:
        assert nbytes > 0, "the shape is meant to be split"
    ws = torch.full((nbytes,), 0xFF, dtype=torch.uint8, device=DEV)     # NaN patterns: only what was written may be read
    out, mass = _call(cache, start, length, q, k, v, ratio, causal, ws)
    ref, ref_mass = _call(cache, start, length, q, k, v, ratio, causal, None)
    if shape in SIXTEEN_BIT_SHAPES and nbytes:
        assert attention_threads(cache, start, length, q, k, v, out.to(q.dtype), causal, workspace=ws) == SIXTEEN_BIT
    assert torch.isfinite(out).all()
    # Either side rounds its probabilities and its output to 16 bits.  Relative to the result a rounding to 8 bits is 2^-9 /
    # sqrt(3) rms, for the terms of a sum of independent values as for the sum; four of them: 2.3e-3.  (What a 32-key tile
    # adds to a row of 2000 keys is 0.13 of it.)
    assert float((out - ref).norm()) <= 1e-2 * float(ref.norm())
    # A single element: the probabilities sum to 1, so their roundings are at most 2^-8 of the largest value, in either call
    assert float((out - ref).abs().max()) <= 2 * 2.0 ** -8 * largest
    # fp32 sums of the same terms in another order; the group-wise kernel sums f16-rounded ones (2^-11 each)
    torch.testing.assert_close(mass, ref_mass, rtol=1e-3, atol=1e-6)


def test_too_small_a_workspace_means_no_split():
    cache = B.Cache(B.make_desc(2, 128, 2, 512, B.KVQ_BF16), DEV)
    x = torch.randn((480, 2, 128), device=DEV).to(torch.bfloat16)
    B.kvq_quantize_append(cache, x, x)
    q = x[:40].contiguous()
    nbytes = B.lib().kvq_attention_workspace_bytes(cache.handle, 0, 480, 40, 40, 1)
    short = torch.full((nbytes - 256,), 0x5A, dtype=torch.uint8, device=DEV)
    out, mass = _call(cache, 0, 480, q, q, q, 1, False, short)
    ref, ref_mass = _call(cache, 0, 480, q, q, q, 1, False, None)
    assert torch.equal(out, ref) and torch.equal(mass, ref_mass)
    assert (short == 0x5A).all()


@pytest.mark.parametrize("bits", [2, 4])
def test_split_call_on_a_flagged_cache_is_served_by_the_vector_kernel(bits):
    """Zero-points beyond the 16-bit kernels' domain: the merge launch computes the call in place of the pieces."""
    heads, tokens, rows = 8, 1500, 1800
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    k = torch.randn((tokens, heads, 128), generator=gen, device=DEV) * 1e-5
    k[..., 0] += 40.0                                  # a large offset after the rotation, a minute range
    k = k.to(torch.bfloat16)
    v, q, cur = (torch.randn((n, heads, 128), generator=gen, device=DEV).to(torch.bfloat16) for n in (tokens, rows, 64))
    cache = B.Cache(B.make_desc(heads, 128, bits, tokens, B.KVQ_BF16), DEV)
    B.kvq_quantize_append(cache, k, v)
    assert float(B.export_all(cache, 0)[2].abs().max()) > 70000.0
    q = q * 0.02
    ws = B._workspace(cache, 0, tokens, rows, 64, 1, None)
    assert ws is not None and attention_threads(cache, 0, tokens, q, cur, cur, torch.empty_like(q), workspace=ws) == SIXTEEN_BIT
    out, mass = torch.empty_like(q), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    ref, ref_mass = torch.empty_like(out), torch.empty_like(mass)
    B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass)
    B.kvq_chunk_attention_fp32(cache, 0, tokens, q, cur, cur, ref, ref_mass)
    torch.cuda.synchronize()
    assert torch.equal(out, ref) and torch.equal(mass, ref_mass)


# Few rows in many pieces; whole rounds with a small remainder: the merge takes 32 and 256 workgroups.
@pytest.mark.parametrize("heads,ratio,tokens,rows,axis", [(2, 2, 4000, 51, 1), (65, 1, 1000, 1024, 0)])
def test_a_flagged_cache_is_served_as_fast_split_as_unsplit(heads, ratio, tokens, rows, axis):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(3)
    k = torch.randn((tokens, heads, 128), generator=gen, device=DEV) * 1e-5
    k[..., 0] += 40.0
    v, q = (torch.randn((n, h, 128), generator=gen, device=DEV).to(torch.bfloat16) for n, h in ((tokens, heads), (rows, heads * ratio)))
    cache = B.Cache(B.make_desc(heads, 128, 2, tokens, B.KVQ_BF16, key_axis=axis), DEV)
    B.kvq_quantize_append(cache, k.to(torch.bfloat16), v)
    assert float(B.export_all(cache, 0, 0, 1)[2].abs().max()) > 65500.0
    q *= 0.02
    nbytes = B.lib().kvq_attention_workspace_bytes(cache.handle, 0, tokens, rows, 0, ratio)
    assert nbytes > 0
    ws, times, results = torch.empty(nbytes, dtype=torch.uint8, device=DEV), {}, {}
    for workspace in (ws, None, ws, None):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        results[workspace is None] = _call(cache, 0, tokens, q, None, None, ratio, False, workspace)
        end.record()
        end.synchronize()
        times[workspace is None] = begin.elapsed_time(end)       # of the second round
    assert torch.equal(results[True][0], results[False][0]) and torch.equal(results[True][1], results[False][1])
    # both run the same rows on the same kernel code; with the grid of the merge alone the split call took 4 and 10 times as long
    assert times[False] < 1.7 * times[True], times


def _c_graph(stream, body):
    """A graph recorded through the HIP runtime, without torch (the library's handle finds the runtime it is linked to)."""
    hip, handle = B.lib(), ctypes.c_void_p(int(stream.cuda_stream))
    graph, executable = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(handle, 0) == 0
    with torch.cuda.stream(stream):
        body()
    assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert hip.hipGraphInstantiate(ctypes.byref(executable), graph, None, None, 0) == 0
    return lambda: hip.hipGraphLaunch(executable, handle)


def test_a_capture_begun_outside_torch_records_no_workspace():
    """The replays of such a graph come at times when torch has given the memory of a work space to other tensors."""
    heads, tokens, rows = 2, 2000, 300
    x, q, cur = (torch.randn((n, heads, 128), device=DEV).to(torch.bfloat16) for n in (tokens, rows, 64))
    cache = B.Cache(B.make_desc(heads, 128, 2, tokens, B.KVQ_BF16), DEV)
    B.kvq_quantize_append(cache, x, x)
    nbytes = B.lib().kvq_attention_workspace_bytes(cache.handle, 0, tokens, rows, 64, 1)
    assert nbytes > 0
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    out, mass = torch.empty_like(q), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass, stream=stream)     # every kernel has run outside a capture
    whole, whole_mass = _call(cache, 0, tokens, q, cur, cur, 1, False, None)
    torch.cuda.synchronize()
    held = torch.cuda.memory_allocated()
    replay = _c_graph(stream, lambda: B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass, stream=stream))
    assert torch.cuda.memory_allocated() == held
    for _ in range(3):
        with torch.cuda.stream(stream):          # takes the memory that a work space of this stream would have had
            others = [torch.full((nbytes,), 0x5A, dtype=torch.uint8, device=DEV) for _ in range(2)]
            out.fill_(float("nan"))
            mass.fill_(float("nan"))
        assert replay() == 0
        torch.cuda.synchronize()
        assert all(bool((o == 0x5A).all()) for o in others)
        assert torch.equal(out.float(), whole) and torch.equal(mass, whole_mass)
        del others


def test_a_capture_by_torch_stays_split():
    heads, tokens, rows = 2, 2000, 300
    x, q, cur = (torch.randn((n, heads, 128), device=DEV).to(torch.bfloat16) for n in (tokens, rows, 64))
    cache = B.Cache(B.make_desc(heads, 128, 2, tokens, B.KVQ_BF16), DEV)
    B.kvq_quantize_append(cache, x, x)
    out, mass = torch.empty_like(q), torch.empty((heads, rows), dtype=torch.float32, device=DEV)
    B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass)
    eager, eager_mass = out.clone(), mass.clone()
    whole_mass = _call(cache, 0, tokens, q, cur, cur, 1, False, None)[1]
    assert not torch.equal(eager_mass, whole_mass)          # the sums run in another order
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.kvq_chunk_attention(cache, 0, tokens, q, cur, cur, out, mass)
    for _ in range(3):
        out.fill_(float("nan"))
        mass.fill_(float("nan"))
        torch.full((1 << 24,), 0x5A, dtype=torch.uint8, device=DEV)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager) and torch.equal(mass, eager_mass)


def test_calls_of_the_vector_kernel_get_no_workspace():
    """More appended blocks than the per-channel kernel lists; the exact correction."""
    heads, rows, block = 2, 300, 64
    cache = B.Cache(B.make_desc(heads, 128, 2, 64 * block, B.KVQ_BF16, key_axis=B.KVQ_KEYS_PER_CHANNEL), DEV)
    x = torch.randn((block, heads, 128), device=DEV).to(torch.bfloat16)
    q = torch.randn((rows, heads, 128), device=DEV).to(torch.bfloat16)
    for blocks in range(1, 42):
        B.kvq_quantize_append(cache, x, x)
        wanted = B.lib().kvq_attention_workspace_bytes(cache.handle, 0, len(cache), rows, 0, 1)
        if blocks >= 30:
            assert (wanted > 0) == (blocks <= 40)
    assert B.lib().kvq_attention_workspace_bytes(cache.handle, block, len(cache) - block, rows, 0, 1) > 0
    per_token = B.Cache(B.make_desc(heads, 128, 2, 2000, B.KVQ_BF16), DEV)
    k = torch.randn((2000, heads, 128), device=DEV).to(torch.bfloat16)
    B.kvq_quantize_append(per_token, k, k)
    out = torch.empty_like(q)
    for correction, grouped, split in [(1, False, True), (2, False, False), (1, True, True), (2, True, False)]:
        torch.cuda.synchronize()
        torch.cuda.reset_peak_memory_stats()
        held = torch.cuda.memory_allocated()
        if grouped:
            B.kvq_chunk_attention_ex(per_token, 0, 2000, q[:8], None, None, out[:8], correction=correction)
        else:
            B.kvq_chunk_attention(per_token, 0, 2000, q[:8], None, None, out[:8], correction=correction)
        assert (torch.cuda.max_memory_allocated() > held) == split
    torch.cuda.synchronize()
