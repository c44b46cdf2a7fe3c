"""GPU parity of kvq_chunk_attention against the CPU oracle (outputs and attention masses).

Where a test over a few hundred rows or keys speaks of the matrix-core kernel of a BF16 / head_dim 128 format, it is the fp32 kernel
that the call runs on; test_gpu_sixteen_bit.py repeats these tests on the 16-bit kernels."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import parity
    return parity


def _cached(w, heads=None):
    from paper_2605_26266_amd import workloads as wl
    ks, vs = zip(*[wl.chunk_kv(w, c, heads) for c in range(w.cached_chunks)])
    return np.concatenate(ks), np.concatenate(vs)


def _fill(P, cache, w):
    from paper_2605_26266_amd import binding as B, workloads as wl
    for c in range(w.cached_chunks):
        k, v = wl.chunk_kv(w, c)
        B.kvq_quantize_append(cache, P.to_dev(k, w.io_dtype), P.to_dev(v, w.io_dtype))


@pytest.mark.parametrize("correction", [1, 0])
@pytest.mark.parametrize("bits", [2, 4])
def test_tiny_fp32(P, bits, correction):
    """Tiny config, fp32 I/O: the fp32 matrix kernel against the double oracle, all rows."""
    import oracle
    from paper_2605_26266_amd import workloads as wl
    w = wl.WORKLOADS["tiny"].with_bits(bits)
    cache = P.make_cache(w, w.cached_tokens)
    _fill(P, cache, w)
    kc, vc = _cached(w)
    kr, vr = wl.chunk_kv(w, w.cached_chunks)
    q = wl.chunk_q(w)
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, correction)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "fp32", correction=correction)
    err = P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_FP32, "tiny")
    print("tiny bits=%d corr=%d: max err %.2e, mean P_S %.4f" % (bits, correction, err, mass.mean()))


@pytest.mark.parametrize("fp32_kernel", [True, False])
@pytest.mark.parametrize("correction", [1, 0])
@pytest.mark.parametrize("bits", [2, 4])
def test_small_all_rows(P, bits, correction, fp32_kernel):
    """Small config in full: 8 heads, 4096 cached + 1024 current tokens, every query row."""
    import oracle
    from paper_2605_26266_amd import workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    cache = P.make_cache(w, w.cached_tokens)
    _fill(P, cache, w)
    kc, vc = _cached(w)
    kr, vr = wl.chunk_kv(w, w.cached_chunks)
    q = wl.chunk_q(w)
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, correction)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", correction=correction, fp32_kernel=fp32_kernel)
    err = P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "small")
    print("small bits=%d corr=%d fp32=%d: max err %.2e" % (bits, correction, fp32_kernel, err))


RAGGED = [
    # (m, cache_start, cache_len, n_cur)
    (1, 0, 1, 0),
    (1, 0, 0, 1),
    (7, 0, 33, 5),
    (64, 3, 61, 64),
    (65, 31, 34, 31),
    (130, 32, 200, 97),
    (257, 5, 1000, 0),
    (300, 0, 0, 333),
    (300, 17, 777, 129),
    (511, 64, 1024, 513),
]


@pytest.mark.parametrize("fp32_kernel", [True, False])
@pytest.mark.parametrize("bits", [2, 4])
def test_ragged_shapes_and_windows(P, bits, fp32_kernel):
    """Row tails, key tails, windows that start and end inside a tile, empty cache, empty current block."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads = 3
    cache = P.make_cache(w, 1100, heads=heads)
    k0, v0 = wl.chunk_kv(w, 0, heads=range(heads))
    k1, v1 = wl.chunk_kv(w, 1, heads=range(heads))
    kc, vc = np.concatenate([k0, k1])[:1100], np.concatenate([v0, v1])[:1100]
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    kr_all, vr_all = wl.chunk_kv(w, 2, heads=range(heads))
    q_all = wl.chunk_q(w, heads=range(heads))
    for (m, start, clen, ncur) in RAGGED:
        q, kr, vr = q_all[:m], kr_all[:ncur], vr_all[:ncur]
        ref, mass_ref, _ = oracle.chunk_attention(q, kc[start:start + clen], vc[start:start + clen], kr, vr, bits, 1)
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", cache_start=start, cache_len=clen,
                                        fp32_kernel=fp32_kernel)
        P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "ragged %s" % ((m, start, clen, ncur),))


def test_softmax_scale_and_large_queries(P):
    """A caller-chosen softmax scale enters the correction squared; big query norms make b matter."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    heads = 2
    cache = P.make_cache(w, 512, heads=heads)
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=512)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=256)
    q = wl.round_to_bf16(wl.chunk_q(w, heads=range(heads))[:256] * np.float32(2.0))
    for sigma in (0.05, 0.125):
        ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 1, sigma=sigma)
        off, mass_off, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 0, sigma=sigma)
        assert np.max(np.abs(mass_ref - mass_off)) > 0.02          # the correction is not a no-op here
        for fp32_kernel in (True, False):
            out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", softmax_scale=sigma, fp32_kernel=fp32_kernel)
            P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "sigma=%g" % sigma)


@pytest.mark.parametrize("bits", [2, 4])
def test_query_dynamic_range(P, bits):
    """Query rows the operand formats of the matrix-core path have to cope with: all zeros, magnitudes far below
    anything a score can see, rows whose rotated vector is one large channel plus small ones (a constant offset
    before the rotation), and a mix of magnitudes over the rows of one 32-row block."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads = 2
    cache = P.make_cache(w, 512, heads=heads)
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=512)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=128)
    q = wl.chunk_q(w, heads=range(heads))[:256].copy()
    rng = np.random.default_rng(77)
    q[0] = 0.0
    q[1] *= np.float32(1e-30)
    q[2] *= np.float32(1e-6)
    q[3:40] = q[3:40] * np.float32(0.5) + np.float32(0.75)        # rotated: one channel of 8.5, the rest small
    q[40:64] *= rng.uniform(0.01, 4.0, size=(24, 1, 1)).astype(np.float32)
    q[64:96, :, 5] += np.float32(6.0)                              # one large raw channel: flat after the rotation
    q = wl.round_to_bf16(q)
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, 1)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16")
    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "dynamic range, %d bits" % bits)


@pytest.mark.parametrize("bits", [2, 4])
def test_large_zero_points(P, bits):
    """Vectors that are a spike in channel 0 plus small noise rotate into a large offset with a small range,
    so their zero-points reach several hundred: beyond one bf16 piece on the matrix-core path."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads = 2
    n_cached, n_cur, m = 200, 64, 96

    def spiky(x, noise):
        x = x * np.float32(noise)
        x[..., 0] += np.float32(2.0)
        return wl.round_to_bf16(x)

    k0, v0 = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    kc, vc = spiky(k0, 2e-3), spiky(v0, 2e-4)
    cache = P.make_cache(w, 256, heads=heads)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    _, _, zeros = B.export_all(cache, 1)
    assert float(zeros.abs().max()) > 300.0                      # the case this test is about
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.chunk_q(w, heads=range(heads))[:m]
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, 1)
    for fp32_kernel in (True, False):
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", fp32_kernel=fp32_kernel)
        P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "large zero-points int%d" % bits)


@pytest.mark.parametrize("bits,group,fp8", [(2, None, False), (4, None, False), (2, 128, True), (2, 32, True)])
def test_zero_points_beyond_the_matrix_core_domain(P, bits, group, fp8):
    """Key vectors with a large offset and a minute range get zero-points of several hundred thousand: beyond
    the 2^16 that the matrix-core kernels carry exactly.  The quantizer marks such a cache and the default entry
    point then serves it with the vector kernel; a cache that is reset and refilled with ordinary vectors goes
    back to the matrix cores.  Both must match the oracle."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads, n_cached, n_cur, m = 2, 200, 64, 96
    k0, v0 = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    kc = k0 * np.float32(1e-5 if not fp8 else 1e-3)
    kc[..., 0] += np.float32(40.0 if not fp8 else 4000.0)     # FP8 steps are at least 2^-9: a larger offset instead
    kc = wl.round_to_bf16(kc)
    vc = v0
    cache = P.make_cache(w, 256, heads=heads, group=group, fp8_meta=fp8)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    P.assert_quantized_equal(cache, kc, vc)
    _, _, zeros = B.export_all(cache, 0)
    assert float(zeros.abs().max()) > 70000.0                    # the case this test is about
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.round_to_bf16(wl.chunk_q(w, heads=range(heads))[:m] * np.float32(0.02 if not fp8 else 2e-4))
    kw = dict(group=group, fp8_meta=fp8) if fp8 else {}
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, 1, **kw)
    for fp32_kernel in (False, True):
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", fp32_kernel=fp32_kernel)
        P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "flagged cache, %s entry" % ("fp32" if fp32_kernel else "default"))
    # reset, ordinary vectors: the flag is cleared by the next append
    B.kvq_cache_reset(cache)
    B.kvq_quantize_append(cache, P.to_dev(k0, "bf16"), P.to_dev(v0, "bf16"))
    q = wl.chunk_q(w, heads=range(heads))[:m]
    ref, mass_ref, _ = oracle.chunk_attention(q, k0, v0, kr, vr, bits, 1, **kw)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16")
    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "after reset")


@pytest.mark.parametrize("bits,group", [(2, 128), (2, 32), (4, 64), (4, 32)])
def test_large_zero_points_fp8_bf16_metadata(P, bits, group):
    """Zero-points beyond +-256 under FP8/BF16 metadata: the stored zero-point is the BF16 rounding of the
    integer one and the codes are taken with the stored value (clamping where that moves them).  Vectors with
    a spike in channel 0 (a DC offset after the rotation) and a tiny range reach them; the value spikes
    alternate in sign and the queries are small, so that the output stays near zero, where BF16 output
    rounding is far inside the bar.  Quantizer bit-exact; the matrix-core kernel of the format (per-token
    kernel for one group per token, group-wise kernel otherwise; INT4 with groups of 32 has none) and the
    vector kernel against the oracle."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads, n_cached, n_cur, m = 2, 300, 64, 96
    k0, v0 = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    kc = k0 * np.float32(1e-3)
    kc[..., 0] += np.float32(8.0)
    vc = v0 * np.float32(1e-3)
    vc[..., 0] += np.where(np.arange(n_cached) % 2 == 0, 8.0, -8.0).astype(np.float32)[:, None]
    kc, vc = wl.round_to_bf16(kc), wl.round_to_bf16(vc)
    cache = P.make_cache(w, 320, heads=heads, group=group, fp8_meta=True)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    P.assert_quantized_equal(cache, kc, vc)
    for which in (0, 1):
        _, _, zeros = B.export_all(cache, which)
        z = zeros.cpu().numpy().astype(np.float64)
        assert np.abs(z).max() > 256.0                         # the case this test is about ...
        assert np.any((np.abs(z) > 256) & (z % 2 == 0))        # ... (BF16 holds even integers only up there)
    # the rounding is visible: the same vectors with fp32 metadata get other zero-points
    _, _, z_plain = oracle.quantize(kc[:, 0, :].astype(np.float64), bits, group, True, False)
    _, _, z_bf16 = oracle.quantize(kc[:, 0, :].astype(np.float64), bits, group, True, True)
    assert np.abs(z_bf16).max() > 256
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.round_to_bf16(wl.chunk_q(w, heads=range(heads))[:m] * np.float32(0.05))
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, 1, group=group, fp8_meta=True)
    for fp32_kernel in (False, True):
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", fp32_kernel=fp32_kernel)
        P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16,
                                 "large BF16 zero-points int%d g%d %s" % (bits, group, "vector" if fp32_kernel else "default"))


@pytest.mark.parametrize("correction", [1, 0])
@pytest.mark.parametrize("bits,group", [(2, 32), (2, 64), (4, 32), (4, 64), (2, 128)])
def test_group_wise_fp8_metadata(P, bits, group, correction):
    """The paper's default storage format: per-group FP8-E4M3 scale and BF16 zero-point; the correction is
    the per-group sum with the group norms of the rotated query (vector kernel)."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads, n_cached, n_cur, m = 2, 1000, 200, 160
    cache = P.make_cache(w, n_cached, heads=heads, group=group, fp8_meta=True)
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.round_to_bf16(wl.chunk_q(w, heads=range(heads))[:m] * np.float32(1.5))
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, correction, group=group, fp8_meta=True)
    for fp32_kernel in (False, True):   # default dispatch (matrix cores where supported) and the vector kernel
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", correction=correction, fp32_kernel=fp32_kernel)
        P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "group %d int%d" % (group, bits))
    if correction:
        off, mass_off, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, 0, group=group, fp8_meta=True)
        assert np.max(np.abs(mass_ref - mass_off)) > 1e-3      # the correction is visible at this size
    # a window inside the cache
    ref, mass_ref, _ = oracle.chunk_attention(q, kc[37:901], vc[37:901], kr, vr, bits, correction, group=group,
                                              fp8_meta=True)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", cache_start=37, cache_len=864, correction=correction)
    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "group %d window" % group)


@pytest.mark.parametrize("group,fp8", [(None, False), (32, True)])
def test_exact_correction_mode(P, group, fp8):
    """correction = 2: the exact log-moment form (Eq. 12) on the vector kernel, against the oracle's; it
    stays within the fourth-order term of the Taylor form."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    heads, n_cached, n_cur, m = 2, 600, 100, 96
    cache = P.make_cache(w, n_cached, heads=heads, group=group, fp8_meta=fp8)
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.round_to_bf16(wl.chunk_q(w, heads=range(heads))[:m] * np.float32(2.0))
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 2, group=group, fp8_meta=fp8)
    tay, mass_tay, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 1, group=group, fp8_meta=fp8)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", correction=2)
    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "exact correction")
    assert 0 < np.max(np.abs(mass_ref - mass_tay)) < 0.05      # the two forms differ, slightly


def _sampled_case(P, name, bits, n_rows, heads, correction=1, cached_chunks=None, group=None):
    """Full-size GPU run as the benchmark launches it; oracle on sampled heads x sampled rows."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS[name].with_bits(bits)
    n_chunks = w.cached_chunks if cached_chunks is None else cached_chunks
    cache = P.make_cache(w, n_chunks * w.chunk_tokens, group=group, fp8_meta=group is not None)
    ks, vs = [], []
    for c in range(n_chunks):
        k, v = wl.chunk_kv(w, c)
        B.kvq_quantize_append(cache, P.to_dev(k, "bf16"), P.to_dev(v, "bf16"))
        ks.append(k[:, heads].copy())
        vs.append(v[:, heads].copy())
    kc, vc = np.concatenate(ks), np.concatenate(vs)
    kr, vr = wl.chunk_kv(w, w.cached_chunks)
    q = wl.chunk_q(w)
    rows = wl.sample_rows(w, n_rows)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", correction=correction)
    ref, mass_ref, _ = oracle.chunk_attention(q[rows][:, heads], kc, vc, kr[:, heads], vr[:, heads], bits, correction,
                                              group=group, fp8_meta=group is not None)
    return P.assert_attention_close(out[rows][:, heads], mass[heads][:, rows], ref, mass_ref, P.TOL_OUT_BF16,
                                    "%s int%d" % (name, bits))


@pytest.mark.parametrize("bits", [2, 4])
def test_mid_sampled_rows(P, bits):
    err = _sampled_case(P, "mid", bits, 48, [0, 23])
    print("mid int%d: max err %.2e" % (bits, err))


@pytest.mark.parametrize("group", [32, 64])
def test_mid_group_wise_sampled_rows(P, group):
    """The paper's default format (INT2, FP8/BF16 metadata per 32 channels) at the mid shape on the matrix
    cores, and g = 64."""
    _sampled_case(P, "mid", 2, 48, [0, 23], group=group)


@pytest.mark.parametrize("group", [64, 32])
def test_mid_group_wise_int4_sampled_rows(P, group):
    """INT4 with FP8/BF16 metadata per 64 or 32 channels at the mid shape on the matrix cores."""
    _sampled_case(P, "mid", 4, 48, [0, 23], group=group)


@pytest.mark.parametrize("correction", [1, 0])
def test_large_sampled_rows(P, correction):
    err = _sampled_case(P, "large", 2, 32, [5, 47], correction)
    print("large corr=%d: max err %.2e" % (correction, err))


def test_stream_append_then_attend(P):
    """Stream config: the same 4096-token chunk is appended t times, each append followed by corrected
    attention from that chunk's queries over the whole cache plus the chunk itself.  Parity on sampled
    heads x rows after 1, 2 and 32 appends (131072 cached tokens at the end)."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["stream"]
    heads = [3, 40]
    cache = P.make_cache(w, w.cached_tokens)
    k, v = wl.chunk_kv(w, 0)
    q = wl.chunk_q(w)
    kd, vd, qd = P.to_dev(k, "bf16"), P.to_dev(v, "bf16"), P.to_dev(q, "bf16")
    out = torch.empty_like(qd)
    mass = torch.empty((w.num_heads, w.chunk_tokens), dtype=torch.float32, device=P.DEV)
    rows = wl.sample_rows(w, 24)
    ks, vs = k[:, heads], v[:, heads]
    for t in range(1, w.cached_chunks + 1):
        B.kvq_quantize_append(cache, kd, vd)
        B.kvq_chunk_attention(cache, 0, len(cache), qd, kd, vd, out, mass, 0.0, 1)
        if t in (1, 2, w.cached_chunks):
            torch.cuda.synchronize()
            got = out.float().cpu().numpy().astype(np.float64)[rows][:, heads]
            got_mass = mass.cpu().numpy().astype(np.float64)[heads][:, rows]
            ref, mass_ref, _ = oracle.chunk_attention(q[rows][:, heads], np.concatenate([ks] * t),
                                                      np.concatenate([vs] * t), ks, vs, 2, 1)
            err = P.assert_attention_close(got, got_mass, ref, mass_ref, P.TOL_OUT_BF16, "stream t=%d" % t)
            print("stream t=%d: max err %.2e, mean P_S %.4f" % (t, err, got_mass.mean()))
    assert len(cache) == w.cached_tokens


@pytest.mark.parametrize("k_mul,v_mul", [(1e-3, 1e3), (30.0, 1e-4), (1.0, 2.0 ** -20)])
def test_extreme_key_and_value_scales(P, k_mul, v_mul):
    """Keys and values far from unit scale: the matrix-core path carries log2(value scale) / key scale inside
    the score accumulators, so tiny key scales and tiny or large value scales are its stress case."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    heads, n_cached, n_cur, m = 2, 300, 64, 128
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    kc, vc = wl.round_to_bf16(kc * np.float32(k_mul)), wl.round_to_bf16(vc * np.float32(v_mul))
    vc[::7] = wl.round_to_bf16(vc[::7] * np.float32(64.0))         # value scales that differ a lot between tokens
    cache = P.make_cache(w, 320, heads=heads)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    P.assert_quantized_equal(cache, kc, vc)
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    kr, vr = wl.round_to_bf16(kr * np.float32(k_mul)), wl.round_to_bf16(vr * np.float32(v_mul))
    q = wl.round_to_bf16(wl.chunk_q(w, heads=range(heads))[:m] * np.float32(min(1.0 / k_mul, 8.0)))
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 1)
    scale = float(np.max(np.abs(ref))) or 1.0
    for fp32_kernel in (True, False):
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", fp32_kernel=fp32_kernel)
        # outputs of magnitude `scale`: the tolerance is the relative one of BF16 outputs
        P.assert_attention_close(out / scale, mass, ref / scale, mass_ref, P.TOL_OUT_BF16,
                                 "k x %g, v x %g" % (k_mul, v_mul))


@pytest.mark.parametrize("bits", [2, 4])
def test_all_zero_vectors_in_the_cache(P, bits):
    """An all-zero key or value vector has scale 0 (Eq. 1 with an empty range): its key scores 0, its value
    contributes nothing, and it still takes its share of the softmax mass.  The matrix-core path carries
    log2(value scale) / key scale in the score, so both scales being 0 is the case to get right."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"].with_bits(bits)
    heads, n_cached, n_cur, m = 2, 160, 48, 96
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    kc, vc = kc.copy(), vc.copy()
    kc[[3, 40, 41, 159]] = 0.0          # zero keys (one of them with a zero value too)
    vc[[5, 40, 100]] = 0.0
    kc[7, 1] = 0.0                      # one head only
    vc[64:96, 0] = 0.0                  # a whole tile of zero values in one head
    cache = P.make_cache(w, 192, heads=heads)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    P.assert_quantized_equal(cache, kc, vc)
    _, scales, _ = B.export_all(cache, 0)
    assert float(scales.min()) == 0.0                             # the case this test is about
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.chunk_q(w, heads=range(heads))[:m]
    for correction in (1, 0):
        ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, bits, correction)
        for fp32_kernel in (True, False):
            out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", correction=correction, fp32_kernel=fp32_kernel)
            P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "zero vectors int%d" % bits)
    # nothing but zero values: the output of the cached part is 0, the mass is not
    vz = np.zeros_like(vc)
    cache2 = P.make_cache(w, 192, heads=heads)
    B.kvq_quantize_append(cache2, P.to_dev(kc, "bf16"), P.to_dev(vz, "bf16"))
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vz, kr, vr, bits, 1)
    out, mass = P.run_gpu_attention(cache2, q, kr, vr, "bf16")
    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "all values zero int%d" % bits)


def test_ring_of_two_tiles(P):
    """The smallest ring the matrix-core loader can meet: two tiles, a window that wraps, stages that reach
    past the window on both sides."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    heads = 2
    cache = P.make_cache(w, 64, heads=heads)
    k, v = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=160)
    q = wl.chunk_q(w, heads=range(heads))[:70]
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=33)
    B.kvq_quantize_append(cache, P.to_dev(k[:64], "bf16"), P.to_dev(v[:64], "bf16"))
    lo = 0
    for step in range(3):
        B.kvq_cache_evict(cache, 32)
        lo += 32
        B.kvq_quantize_append(cache, P.to_dev(k[lo + 32:lo + 64], "bf16"), P.to_dev(v[lo + 32:lo + 64], "bf16"))
        kc, vc = k[lo:lo + 64], v[lo:lo + 64]
        P.assert_quantized_equal(cache, kc, vc)
        for (start, clen) in ((0, 64), (5, 50), (33, 31)):
            ref, mass_ref, _ = oracle.chunk_attention(q, kc[start:start + clen], vc[start:start + clen], kr, vr, 2, 1)
            for fp32_kernel in (False, True):
                out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", cache_start=start, cache_len=clen,
                                                fp32_kernel=fp32_kernel)
                P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "two-tile ring, step %d" % step)


@pytest.mark.parametrize("group,fp8", [(None, False), (32, True)])
def test_sliding_window_ring(P, group, fp8):
    """A cache with room for three 96-token chunks slides over nine chunks: evict the oldest, append the
    next, attend to the window.  After the storage has wrapped, codes and attention still equal the
    oracle's on the same logical window, for windows that start and end inside tiles too."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    heads, chunk, window = 2, 96, 3
    cache = P.make_cache(w, chunk * window, heads=heads, group=group, fp8_meta=fp8)
    chunks = [wl.chunk_kv(w, c, heads=range(heads), n_tokens=chunk) for c in range(9)]
    q = wl.chunk_q(w, heads=range(heads))[:80]
    kr, vr = wl.chunk_kv(w, 20, heads=range(heads), n_tokens=40)
    live = []
    for c, (k, v) in enumerate(chunks):
        if len(live) == window:
            B.kvq_cache_evict(cache, chunk)
            live.pop(0)
        B.kvq_quantize_append(cache, P.to_dev(k, "bf16"), P.to_dev(v, "bf16"))
        live.append((k, v))
        assert len(cache) == chunk * len(live)
        if c in (2, 4, 5, 8):
            kc, vc = np.concatenate([x[0] for x in live]), np.concatenate([x[1] for x in live])
            P.assert_quantized_equal(cache, kc, vc)
            for (start, clen) in ((0, len(kc)), (17, len(kc) - 40)):
                ref, mass_ref, _ = oracle.chunk_attention(q, kc[start:start + clen], vc[start:start + clen], kr, vr, 2, 1,
                                                          group=group, fp8_meta=fp8)
                for fp32_kernel in (False, True):
                    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", cache_start=start, cache_len=clen,
                                                    fp32_kernel=fp32_kernel)
                    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "ring chunk %d" % c)
    # evictions that are not multiples of a tile: the next append must not touch a tile that is still live
    B.kvq_cache_evict(cache, 50)
    with pytest.raises(B.KvqError) as e:
        B.kvq_quantize_append(cache, P.to_dev(chunks[0][0][:50], "bf16"), P.to_dev(chunks[0][1][:50], "bf16"))
    assert e.value.status == B.KVQ_ERR_CAPACITY
    B.kvq_quantize_append(cache, P.to_dev(chunks[0][0][:32], "bf16"), P.to_dev(chunks[0][1][:32], "bf16"))
    kc = np.concatenate([live[0][0][50:], live[1][0], live[2][0], chunks[0][0][:32]])
    vc = np.concatenate([live[0][1][50:], live[1][1], live[2][1], chunks[0][1][:32]])
    P.assert_quantized_equal(cache, kc, vc)
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 1, group=group, fp8_meta=fp8)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16")
    P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16, "ring, ragged eviction")


def test_seeded_sweep_of_rings_and_windows(P):
    """Forty seeded cases: ring capacities from 2 to 20 tiles, random evictions and appends (the storage wraps),
    every cache format the matrix-core kernels serve, random windows, row counts, current-block sizes."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    rng = np.random.default_rng(7)
    checked = 0
    for case in range(40):
        bits = int(rng.choice([2, 4]))
        group, fp8 = [(None, False), (128, True), (32, True), (64, True)][int(rng.integers(0, 4))]
        w = wl.WORKLOADS["small"].with_bits(bits)
        heads = int(rng.integers(1, 4))
        cap = 32 * int(rng.integers(2, 21))
        cache = P.make_cache(w, cap, heads=heads, group=group, fp8_meta=fp8)
        src_k, src_v = wl.chunk_kv(w, case % 4, heads=range(heads), n_tokens=1024)
        live_k, live_v, pos = [], [], 0
        for _ in range(int(rng.integers(1, 7))):
            if live_k and rng.random() < 0.7:
                ev = min(len(live_k), 32 * int(rng.integers(1, 6)))
                B.kvq_cache_evict(cache, ev)
                live_k, live_v = live_k[ev:], live_v[ev:]
            room = cap - len(live_k)
            n_app = int(rng.integers(1, room + 1)) if room > 0 else 0
            if n_app == 0 or pos + n_app > 1024:
                continue
            try:
                B.kvq_quantize_append(cache, P.to_dev(src_k[pos:pos + n_app], "bf16"), P.to_dev(src_v[pos:pos + n_app], "bf16"))
            except B.KvqError as e:        # the append would touch a tile that is still live
                assert e.status == B.KVQ_ERR_CAPACITY
                continue
            live_k += list(src_k[pos:pos + n_app])
            live_v += list(src_v[pos:pos + n_app])
            pos += n_app
        assert len(cache) == len(live_k)
        if not live_k:
            cache.close()
            continue
        kc, vc = np.stack(live_k), np.stack(live_v)
        m, ncur = int(rng.integers(1, 600)), int(rng.integers(0, 100))
        start = int(rng.integers(0, len(kc)))
        clen = int(rng.integers(1, len(kc) - start + 1))
        corr = int(rng.integers(0, 2))
        q = wl.chunk_q(w, heads=range(heads))[:m]
        kr, vr = wl.chunk_kv(w, 5, heads=range(heads), n_tokens=max(ncur, 1))
        kr, vr = kr[:ncur], vr[:ncur]
        kw = dict(group=group, fp8_meta=True) if fp8 else {}
        ref, mass_ref, _ = oracle.chunk_attention(q, kc[start:start + clen], vc[start:start + clen], kr, vr, bits, corr, **kw)
        out, mass = P.run_gpu_attention(cache, q, kr, vr, "bf16", cache_start=start, cache_len=clen, correction=corr)
        P.assert_attention_close(out, mass, ref, mass_ref, P.TOL_OUT_BF16,
                                 "case %d: int%d group %s fp8 %s heads %d cap %d live %d window (%d, %d) m %d cur %d corr %d"
                                 % (case, bits, group, fp8, heads, cap, len(kc), start, clen, m, ncur, corr))
        checked += 1
        cache.close()
    assert checked >= 30


@pytest.mark.parametrize("io,group,fp8", [("bf16", None, False), ("bf16", 32, True), ("fp32", None, False)])
@pytest.mark.parametrize("causal", [False, True])
def test_grouped_query_heads_and_causal_block(P, io, group, fp8, causal):
    """Partial-prefill shape: 6 query heads over 2 key/value heads, the current block causal.  Runs the
    fp32 matrix kernel on both I/O types (longer causal calls: test_gpu_sixteen_bit.py)."""
    import oracle
    from dataclasses import replace
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = replace(wl.WORKLOADS["small"], io_dtype=io)
    kv_heads, ratio, n_cached = 2, 3, 500
    cache = P.make_cache(w, n_cached, heads=kv_heads, group=group, fp8_meta=fp8)
    kc, vc = wl.chunk_kv(w, 0, heads=range(kv_heads), n_tokens=n_cached)
    B.kvq_quantize_append(cache, P.to_dev(kc, io), P.to_dev(vc, io))
    q_all = wl.chunk_q(w, heads=range(kv_heads * ratio))
    tol = P.TOL_OUT_BF16 if io == "bf16" else P.TOL_OUT_FP32
    for (m, n_cur) in ((300, 300), (70, 333), (1, 64)):      # several row blocks; queries = tail of the block; one query
        kr, vr = wl.chunk_kv(w, 1, heads=range(kv_heads), n_tokens=n_cur)
        q = q_all[:m]
        ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 1, group=group, fp8_meta=fp8, causal=causal)
        out, mass = P.run_gpu_attention(cache, q, kr, vr, io, causal=causal)
        P.assert_attention_close(out, mass, ref, mass_ref, tol, "gqa causal=%s m=%d n=%d" % (causal, m, n_cur),
                                 mass_floor=1e-4 if causal else None)
    # no cached keys at all: pure causal self-attention of the block
    kr, vr = wl.chunk_kv(w, 1, heads=range(kv_heads), n_tokens=96)
    q = q_all[:96]
    ref, mass_ref, _ = oracle.chunk_attention(q, kc[:0], vc[:0], kr, vr, 2, 1, group=group, fp8_meta=fp8, causal=causal)
    out, mass = P.run_gpu_attention(cache, q, kr, vr, io, cache_len=0, causal=causal)
    P.assert_attention_close(out, mass, ref, mass_ref, tol, "gqa no cache", mass_floor=1e-4 if causal else None)
    with pytest.raises(B.KvqError):      # causal needs the queries to be the tail of the current block
        P.run_gpu_attention(cache, q_all[:100], kr, vr, io, causal=True)


@pytest.mark.parametrize("name,io,group,fp8", [("small", "bf16", None, False), ("small", "bf16", 32, True),
                                               ("small", "bf16", 64, True), ("small", "fp32", None, False),
                                               ("tiny", "fp32", None, False)])
def test_randomised_rotation_signs(P, name, io, group, fp8):
    """Sign vector of the randomised Hadamard rotation on every kernel: the quantize kernels (head_dim 128
    and generic), the per-token and group-wise matrix-core attention kernels and the vector kernel."""
    import oracle
    from dataclasses import replace
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = replace(wl.WORKLOADS[name], io_dtype=io)
    d, heads, n_cached = w.head_dim, min(2, w.num_heads), min(333, w.chunk_tokens - 3)
    rng = np.random.default_rng(77)
    negate = rng.random(d) < 0.5
    signs = np.where(negate, -1.0, 1.0)
    cache = P.make_cache(w, n_cached + 64, heads=heads, group=group, fp8_meta=fp8)
    B.kvq_cache_set_rotation_signs(cache, negate)
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    B.kvq_quantize_append(cache, P.to_dev(kc, io), P.to_dev(vc, io))
    P.assert_quantized_equal(cache, kc, vc, signs=signs)
    with pytest.raises(B.KvqError):                       # stored codes belong to the rotation they were written with
        B.kvq_cache_set_rotation_signs(cache, None)
    q = wl.chunk_q(w, heads=range(heads))[:150]
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=min(70, w.chunk_tokens))
    tol = P.TOL_OUT_BF16 if io == "bf16" else P.TOL_OUT_FP32
    for correction in (0, 1):
        ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, w.bits, correction, group=group, fp8_meta=fp8,
                                                  signs=signs)
        out, mass = P.run_gpu_attention(cache, q, kr, vr, io, correction=correction)
        P.assert_attention_close(out, mass, ref, mass_ref, tol, "signs, correction %d" % correction)
    ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr[:0], vr[:0], w.bits, 1, group=group, fp8_meta=fp8, signs=signs)
    out, mass = P.run_gpu_attention(cache, q, None, None, io)
    P.assert_attention_close(out, mass, ref, mass_ref, tol, "signs, cache only")
    # back to the plain rotation on the emptied cache
    B.kvq_cache_reset(cache)
    B.kvq_cache_set_rotation_signs(cache, None)
    B.kvq_quantize_append(cache, P.to_dev(kc, io), P.to_dev(vc, io))
    P.assert_quantized_equal(cache, kc, vc)


def test_argument_errors(P):
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    cache = P.make_cache(w, 64)
    k, v = wl.chunk_kv(w, 0, n_tokens=64)
    B.kvq_quantize_append(cache, P.to_dev(k, "bf16"), P.to_dev(v, "bf16"))
    q = P.to_dev(wl.chunk_q(w)[:16], "bf16")
    out = torch.empty_like(q)
    with pytest.raises(B.KvqError) as e:
        B.kvq_chunk_attention(cache, 0, 65, q, None, None, out)      # window beyond the cache
    assert e.value.status == B.KVQ_ERR_INVALID_ARG
    with pytest.raises(B.KvqError):
        B.kvq_chunk_attention(cache, 0, 0, q, None, None, out)       # no keys at all
    with pytest.raises(B.KvqError):
        B.kvq_chunk_attention(cache, 0, 64, q, None, None, q)        # out aliases q
    with pytest.raises(B.KvqError):
        B.kvq_chunk_attention(cache, 0, 64, q, None, None, out, correction=3)
    B.kvq_chunk_attention(cache, 0, 64, q[:0], None, None, out[:0])   # m == 0 is a no-op


@pytest.mark.parametrize("name,io,bits,group,fp8", [("small", "bf16", 2, None, False), ("small", "bf16", 4, 32, True),
                                                    ("tiny", "fp32", 2, None, False)])
def test_attention_diagnostics(P, name, io, bits, group, fp8):
    """kvq_attention_diagnostics against the oracle: both cached masses to the bar of P_S, the divergence and
    the output MSE to 2e-3 relative (they are sums of squares of small differences taken in fp32)."""
    import oracle
    from dataclasses import replace
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = replace(wl.WORKLOADS[name], io_dtype=io, bits=bits)
    heads = min(2, w.num_heads)
    n_cached, n_cur, m = min(300, w.chunk_tokens), min(150, w.chunk_tokens), min(70, w.chunk_tokens)
    cache = P.make_cache(w, n_cached + 40, heads=heads, group=group, fp8_meta=fp8)
    pad_k, pad_v = wl.chunk_kv(w, 2, heads=range(heads), n_tokens=40)      # the window starts inside a tile
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    B.kvq_quantize_append(cache, P.to_dev(pad_k, io), P.to_dev(pad_v, io))
    B.kvq_quantize_append(cache, P.to_dev(kc, io), P.to_dev(vc, io))
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    q = wl.chunk_q(w, heads=range(heads))[:m]
    qd, kcd, vcd, krd, vrd = (P.to_dev(x, io) for x in (q, kc, vc, kr, vr))
    for correction in (0, 1, 2):
        diag = torch.full((heads, m, 4), float("nan"), dtype=torch.float32, device=P.DEV)
        B.kvq_attention_diagnostics(cache, 40, n_cached, qd, kcd, vcd, krd, vrd, diag, correction=correction)
        torch.cuda.synchronize()
        got = diag.cpu().numpy().astype(np.float64)
        ref = oracle.chunk_diagnostics(q, kc, vc, kr, vr, bits, correction, group=group, fp8_meta=fp8)
        assert np.all(np.isfinite(got))
        for col, name_ in ((0, "P_S unquantized"), (1, "P_S quantized")):
            for g_, r_ in ((got[:, :, col], ref[:, :, col]), (1 - got[:, :, col], 1 - ref[:, :, col])):
                sel = r_ >= 1e-4
                assert np.max(np.abs(g_[sel] - r_[sel]) / r_[sel]) <= P.TOL_MASS_REL, name_
        for col, name_ in ((2, "JSD"), (3, "MSE")):
            err = np.abs(got[:, :, col] - ref[:, :, col])
            assert np.all(err <= 2e-3 * ref[:, :, col] + 1e-9), "%s: %.3e" % (name_, float(np.max(err / (ref[:, :, col] + 1e-30))))
    # the quantized side is what kvq_chunk_attention reports
    out, mass = P.run_gpu_attention(cache, q, kr, vr, io, cache_start=40, cache_len=n_cached, correction=2, fp32_kernel=True)
    assert np.allclose(mass, got[:, :, 1], rtol=1e-5, atol=1e-7)
    # no current block, and no cached window
    diag = torch.full((heads, m, 4), float("nan"), dtype=torch.float32, device=P.DEV)
    B.kvq_attention_diagnostics(cache, 40, n_cached, qd, kcd, vcd, None, None, diag)
    torch.cuda.synchronize()
    ref = oracle.chunk_diagnostics(q, kc, vc, kr[:0], vr[:0], bits, 1, group=group, fp8_meta=fp8)
    got = diag.cpu().numpy().astype(np.float64)
    assert np.allclose(got[:, :, :2], 1.0, atol=1e-6)
    assert np.all(np.abs(got[:, :, 2:] - ref[:, :, 2:]) <= 2e-3 * ref[:, :, 2:] + 1e-9)
    B.kvq_attention_diagnostics(cache, 0, 0, qd, None, None, krd, vrd, diag)
    torch.cuda.synchronize()
    got = diag.cpu().numpy()
    assert np.all(got[:, :, :2] == 0.0) and np.all(np.abs(got[:, :, 2:]) <= 1e-9)


def test_attention_replayed_from_a_graph(P):
    """The launching calls only enqueue kernels on the stream they are given (no memset, no host synchronisation;
    the work space of a split call comes from the graph's own pool), so a serving loop can capture them: a captured quantize-free step (attention
    over a filled cache) is replayed three times with new queries, eager work in between, and every replay
    must equal the eager result bit for bit and the oracle to the usual bar."""
    import oracle
    from paper_2605_26266_amd import binding as B, workloads as wl
    w = wl.WORKLOADS["small"]
    heads, n_cached, n_cur, m = 2, 700, 130, 300
    cache = P.make_cache(w, n_cached, heads=heads)
    kc, vc = wl.chunk_kv(w, 0, heads=range(heads), n_tokens=n_cached)
    B.kvq_quantize_append(cache, P.to_dev(kc, "bf16"), P.to_dev(vc, "bf16"))
    kr, vr = wl.chunk_kv(w, 1, heads=range(heads), n_tokens=n_cur)
    krd, vrd = P.to_dev(kr, "bf16"), P.to_dev(vr, "bf16")
    q_all = wl.chunk_q(w, heads=range(heads))
    qd = P.to_dev(q_all[:m], "bf16")
    out = torch.empty_like(qd)
    mass = torch.empty((heads, m), dtype=torch.float32, device=P.DEV)
    B.kvq_chunk_attention(cache, 0, n_cached, qd, krd, vrd, out, mass)      # first launch outside the capture
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.kvq_chunk_attention(cache, 0, n_cached, qd, krd, vrd, out, mass)
    for rep in range(3):
        q = q_all[rep * 100:rep * 100 + m]
        qd.copy_(P.to_dev(q, "bf16"))
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        got, got_mass = out.float().cpu().numpy().astype(np.float64), mass.cpu().numpy().astype(np.float64)
        eager_out, eager_mass = torch.empty_like(qd), torch.empty_like(mass)
        B.kvq_chunk_attention(cache, 0, n_cached, qd, krd, vrd, eager_out, eager_mass)
        torch.cuda.synchronize()
        assert torch.equal(eager_out, out) and torch.equal(eager_mass, mass), "replay %d differs from the eager call" % rep
        ref, mass_ref, _ = oracle.chunk_attention(q, kc, vc, kr, vr, 2, 1)
        P.assert_attention_close(got, got_mass, ref, mass_ref, P.TOL_OUT_BF16, "graph replay %d" % rep)
