"""Host side of the split key ranges: work space sizes and argument checks (no kernel runs: the cache is empty)."""
import ctypes

import pytest

from paper_2605_26266_amd import binding as B

FAKE = 0x10000000


def _cache(*args, **kw):
    desc = B.make_desc(*args, **kw)
    handle = ctypes.c_void_p()
    assert B.lib().kvq_cache_create(ctypes.byref(desc), FAKE, B.kvq_cache_bytes(desc), ctypes.byref(handle)) == B.KVQ_OK
    return handle


def _bytes(handle, rows, current, ratio=1, start=0, cached=0):
    return B.lib().kvq_attention_workspace_bytes(handle, start, cached, rows, current, ratio)


@pytest.mark.parametrize("heads,rows,current,ratio,split", [
    (8, 1024, 5120, 1, True),       # 32 blocks of 256 rows
    (1, 1, 64, 1, False),           # two tiles: nothing to divide
    (64, 1024, 5120, 1, False),     # 256 blocks: exactly one round
    (8, 1, 8192, 4, True),          # a row per query head
])
def test_work_space_is_asked_for_where_a_call_is_split(heads, rows, current, ratio, split):
    h = _cache(heads, 128, 2, 1024)
    n = _bytes(h, rows, current, ratio)
    assert (n > 0) == split
    # every piece holds 32-row blocks of head_dim + 4 floats per row; at most 2048 pieces of 256 rows
    assert n % (32 * 132 * 4) == 0 and n <= 2048 * 256 * 132 * 4
    B.lib().kvq_cache_destroy(h)


def test_calls_that_are_never_split_and_invalid_ones_need_none():
    per_channel = _cache(8, 64, 2, 1024, key_axis=B.KVQ_KEYS_PER_CHANNEL)     # vector kernel
    assert _bytes(per_channel, 1024, 5120) == 0
    no_cached_keys = _cache(8, 128, 2, 1024, key_axis=B.KVQ_KEYS_PER_CHANNEL)           # vector kernel
    assert _bytes(no_cached_keys, 1024, 5120) == 0
    B.lib().kvq_cache_destroy(no_cached_keys)
    long_ring = _cache(8, 128, 2, 1 << 25)                                              # vector kernel
    assert _bytes(long_ring, 1024, 5120) == 0
    B.lib().kvq_cache_destroy(long_ring)
    h = _cache(8, 128, 2, 1024)
    for bad in [dict(rows=0, current=64), dict(rows=64, current=-1), dict(rows=64, current=64, ratio=0),
                dict(rows=64, current=64, ratio=65), dict(rows=64, current=64, cached=1), dict(rows=64, current=64, start=-1)]:
        assert _bytes(h, **bad) == 0
    assert B.lib().kvq_attention_workspace_bytes(None, 0, 0, 64, 64, 1) == 0
    ws = B.lib().kvq_chunk_attention_ws
    for pointer, size in [(FAKE + 16, 256), (None, 256)]:      # misaligned; bytes without memory
        assert ws(h, 0, 0, FAKE, FAKE, FAKE, 64, 64, 1024, 128, 0.0, 1, None, FAKE + (1 << 20), None, pointer, size, None) \
            == B.KVQ_ERR_INVALID_ARG
    B.lib().kvq_cache_destroy(per_channel)
    B.lib().kvq_cache_destroy(h)


@pytest.mark.parametrize("args", [(128, 2, B.KVQ_BF16, None, B.KVQ_META_FP32), (128, 4, B.KVQ_BF16, 32, B.KVQ_META_FP8_BF16),
                                  (64, 2, B.KVQ_BF16, None, B.KVQ_META_FP32), (128, 4, B.KVQ_FP32, 64, B.KVQ_META_FP8_BF16)])
def test_calls_the_binding_does_not_ask_about_are_not_split(args):
    dim, bits, io, group, meta = args
    for heads in (1, 3, 8, 31, 64):
        h = _cache(heads, dim, bits, 1024, io_dtype=io, group_size=group, meta_format=meta)
        for rows in (1, 5, 32, 33, 256, 300, 1024, 5000):
            for current in (1, 64, 250, B._NEVER_SPLIT_KEYS):
                for ratio in (1, 4, 64):
                    # two tiles more than the keys fill: a cached window may begin and end inside a tile
                    assert _bytes(h, rows, current, ratio) == 0 and _bytes(h, rows, current + 64, ratio) == 0
        B.lib().kvq_cache_destroy(h)


def test_grids_beyond_the_launch_limit_go_to_the_vector_kernel():
    """A grid has fewer than 2^32 threads.  The fp32 kernel has 512 for 32 rows, the vector kernel 64 or 128 for one row of one
    head of its second grid dimension: 268 heads x 1003552 rows are 8404748 units, too many for the former only."""
    h = _cache(268, 64, 2, 1024)
    assert _bytes(h, 31233 * 32, 5120) > 0          # 8370444 units, the last 12 split
    assert _bytes(h, 31361 * 32, 5120) == 0
    B.lib().kvq_cache_destroy(h)
