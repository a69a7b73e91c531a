"""The paths of the stratified and systematic schemes give the same bits: one
workgroup per vector or segment (up to 1024, 4096 and 16384 weights), one block
per workgroup with its own carries, and records, carries and one block per
wave, at the edges of their ranges; and the resolve pass over a sorted
ancestry, inside and outside its LDS window, is Code 10."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import inputs
from test_gpu_parity import dev, host, new_flags, pfr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SCHEMES = ("stratified", "systematic")
GENERAL = {"single_wg_max": 0, "direct_max_blocks": 0, "batch_scan_wg_max_len": 0}


def general(scheme, w, **kw):
    """The result of records, carries and one block per wave."""
    m = pfr()
    saved = m.get_tuning()
    try:
        m.set_tuning(**GENERAL)
        return host(getattr(m, "resample_" + scheme)(w, **kw))
    finally:
        m.set_tuning(**saved)


def weights(kind, n, dtype):
    g = np.random.default_rng(n)
    if kind == "wide":  # blocks 2^40 apart, zeros, a run of zero blocks
        w = np.ldexp(g.random(n) + 0.5, g.integers(-20, 20, n))
        w *= np.ldexp(1.0, g.integers(-20, 20, (n + 1023) // 1024)).repeat(1024)[:n]
        w[g.random(n) < 0.3] = 0
        w[n // 3:n // 2] = 0
        if not w.any():
            w[0] = 1
        return w.astype(dtype)
    if kind == "one":  # all the mass on one weight
        w = np.zeros(n, dtype)
        w[n // 2] = 3
        return w
    return inputs.weights(n, kind, seed=n, dtype=dtype)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 5, 1023, 1024, 1025, 4095, 4096, 4097, 70001, 262144, 262145,
                               524289, 1048575, 1048576, 1048577])
def test_single_vector_paths_agree(n, dtype):
    for kind in (0.0, 4.0, "wide", "one"):
        w = dev(weights(kind, n, dtype))
        for s in SCHEMES:
            a = host(getattr(pfr(), "resample_" + s)(w, seed=7, offset=n & 3, filter_base=2))
            ref = general(s, w, seed=7, offset=n & 3, filter_base=2)
            assert np.array_equal(a, ref), (kind, s)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 5, 1022, 1023, 1024, 1025, 2047, 2048, 4097, 70001, 262143,
                               524289, 1048575, 1048576, 1048577])
def test_multinomial_paths_agree(n, dtype):
    """One block per workgroup (up to 1024 blocks) against records, carries and
    one block per wave: one weight over every exponential block, blocks without
    weight, ranges within one exponential block."""
    m = pfr()
    saved = m.get_tuning()
    for kind in (0.0, 4.0, "wide", "one"):
        w = dev(weights(kind, n, dtype))
        ref = general("multinomial", w, seed=7, offset=n & 3, filter_base=2)
        try:
            m.set_tuning(single_wg_max=0, direct_max_blocks=1024)
            a = host(m.resample_multinomial(w, seed=7, offset=n & 3, filter_base=2))
            b = host(m.resample_permuted("multinomial", w, seed=7, offset=n & 3, filter_base=2)[0])
        finally:
            m.set_tuning(**saved)
        assert np.array_equal(a, ref) and np.array_equal(b, ref), kind


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("filters", [3, 40])
@pytest.mark.parametrize("with_max_len", [True, False])
def test_segment_tiers_agree_with_single_calls(filters, dtype, with_max_len):
    sizes = ([1, 0, 1024, 1025, 3, 4096, 4097, 16384, 1000, 16383, 2049] * 4)[:filters]
    if filters == 40:
        sizes += [1] * 300  # more segments than one round of workgroups
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    kinds = [0.0, 4.0, "wide", "one", 2.0]
    w = np.concatenate([weights(kinds[f % 5], n, dtype) if n else np.zeros(0, dtype)
                        for f, n in enumerate(sizes)])
    for s in SCHEMES:
        a = host(getattr(pfr(), "resample_" + s)(dev(w), seed=3, filter_base=1, offsets=dev(off),
                                                 max_len=max(sizes) if with_max_len else None))
        for f, n in enumerate(sizes):
            if n:
                ref = general(s, dev(w[off[f]:off[f + 1]]), seed=3, filter_base=1 + f)
                assert np.array_equal(a[off[f]:off[f + 1]], ref), (s, f, n)


def test_bad_and_zero_segments_give_the_identity():
    sizes = [1000, 4000, 16000, 300, 5000]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = np.concatenate([weights(1.0, n, np.float32) for n in sizes])
    w[10] = np.nan
    w[off[1]:off[2]] = 0
    w[off[3] - 1] = -1
    for s in SCHEMES:
        fl = new_flags()
        a = host(getattr(pfr(), "resample_" + s)(dev(w), offsets=dev(off), max_len=16000, flags=fl))
        for f in (0, 1, 2):
            assert np.array_equal(a[off[f]:off[f + 1]], np.arange(sizes[f])), f
        for f in (3, 4):
            ref = general(s, dev(w[off[f]:off[f + 1]]), filter_base=f)
            assert np.array_equal(a[off[f]:off[f + 1]], ref), f
        m = pfr()
        assert int(host(fl)[0]) == m.FLAG_BAD_WEIGHTS | m.FLAG_ZERO_TOTAL


@pytest.mark.parametrize("scheme", ["stratified", "systematic", "multinomial"])
@pytest.mark.parametrize("n", [4097, 8191, 8192, 65537, 1 << 20, (1 << 21) - 1, 1 << 21,
                               (1 << 21) + 1])
def test_resolve_of_the_fused_claim(scheme, n):
    """The fused permutation of sorted ancestries whose chains stay near their
    start, drift out of the window, or do not move."""
    g = np.random.default_rng(3)
    half = np.where(np.arange(n) < n // 2, 0.01, 1.0)  # drifts by n / 2
    for w in (inputs.weights(n, 0.0, seed=1), inputs.weights(n, 3.0, seed=2),
              (half * (g.random(n) + 0.5)).astype(np.float32), np.ones(n, np.float32),
              np.zeros(n, np.float32)):
        a, c = pfr().resample_permuted(scheme, dev(w), seed=5)
        a, c = host(a), host(c)
        assert np.array_equal(c, oracle.permute(a)[0])


@pytest.mark.parametrize("scheme", ["stratified", "systematic", "multinomial"])
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("short", [0, 6000])
def test_permutation_fused_into_a_batch(scheme, dtype, short):
    """Tiles of 4096 slots at their edges, empty segments, chains that leave
    the window, invalid and zero segments; and (short) segments so small that
    the claims do not fit, which are permuted after the emission as before."""
    sizes = [0, 1, 4095, 4096, 4097, 0, 31, 8191, 8192, 8193, 16385, 65537, 200000, 3, 12288, 5000]
    sizes += [1, 0, 2] * (short // 3) + [0]
    kinds = [0.0, 4.0, "wide", "one", 2.0]
    ws = [weights(kinds[f % 5], n, dtype) if n else np.zeros(0, dtype) for f, n in enumerate(sizes)]
    g = np.random.default_rng(1)
    ws[12] = (np.where(np.arange(200000) < 100000, 0.01, 1.0) * (g.random(200000) + 0.5)).astype(dtype)
    ws[14][5] = np.nan
    ws[15][:] = 0
    if short:  # mostly tiny segments
        for f in (11, 12):
            sizes[f], ws[f] = 7, ws[f][:7]
    w, off = np.concatenate(ws), np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    fl = new_flags()
    kw = dict(seed=3, filter_base=1, offsets=dev(off))
    a, c = pfr().resample_permuted(scheme, dev(w), flags=fl, **kw)
    a, c = host(a), host(c)
    assert np.array_equal(a, host(getattr(pfr(), "resample_" + scheme)(dev(w), **kw)))
    for f, n in enumerate(sizes):
        if n:
            s = slice(off[f], off[f + 1])
            assert np.array_equal(c[s], oracle.permute(a[s])[0]), (f, n)
    m = pfr()
    assert int(host(fl)[0]) == m.FLAG_BAD_WEIGHTS | m.FLAG_ZERO_TOTAL


@pytest.mark.parametrize("scheme", SCHEMES)
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("max_len", [1024, 4096, 16384])
def test_permutation_in_one_workgroup(scheme, dtype, max_len):
    """Segments of every tier with the permutation in the same launch, chains
    long enough for the list and past its end, invalid and zero segments; and
    single vectors."""
    sizes = [n for n in (1, 0, 2, 5, 255, 1023, 1024, 1025, 4095, 4096, 4097, 9000, 16383, 16384)
             if n <= max_len] * 3
    kinds = [0.0, 4.0, "wide", "one", "drift"]
    ws = []
    for f, n in enumerate(sizes):
        k = kinds[f % 5]
        ws.append(np.linspace(0.01, 1.0, n).astype(dtype) if k == "drift" else
                  weights(k, n, dtype) if n else np.zeros(0, dtype))
    ws[4][:] = 0
    ws[5][3] = np.inf
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = dev(np.concatenate(ws))
    fl = new_flags()
    kw = dict(seed=3, filter_base=1, offsets=dev(off), max_len=max_len)
    a, c = pfr().resample_permuted(scheme, w, flags=fl, **kw)
    a, c = host(a), host(c)
    assert np.array_equal(a, host(getattr(pfr(), "resample_" + scheme)(w, **kw)))
    for f, n in enumerate(sizes):
        if n:
            s = slice(off[f], off[f + 1])
            assert np.array_equal(c[s], oracle.permute(a[s])[0]), (f, n)
            if n <= 4096:
                a1, c1 = pfr().resample_permuted(scheme, dev(ws[f]), seed=3, filter_base=1 + f)
                assert np.array_equal(host(a1), a[s]) and np.array_equal(host(c1), c[s]), (f, n)
    m = pfr()
    assert int(host(fl)[0]) == m.FLAG_BAD_WEIGHTS | m.FLAG_ZERO_TOTAL


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [1, 2, 10, 1022, 1023, 1024, 2049, 4095, 4096])
def test_short_multinomial_with_and_without_workspace(dtype, n):
    """Two launches with a workspace, one workgroup without; blocks so far
    apart that the carries' truncation shows; and with the permutation."""
    m = pfr()
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    apart = np.ldexp(1.0, -30 * (np.arange(n) // 1024)) * np.random.default_rng(n).random(n)
    for w in ([weights(k, n, dtype) for k in (0.0, 4.0, "wide", "one")] +
              [apart.astype(dtype), np.zeros(n, dtype)]):
        w = dev(w)
        fl, fl0 = new_flags(), new_flags()
        a = host(m.resample_multinomial(w, seed=4, offset=1, filter_base=3, flags=fl))
        b = host(m.resample_multinomial(w, seed=4, offset=1, filter_base=3, flags=fl0,
                                        workspace=none))
        assert np.array_equal(a, b) and int(host(fl)[0]) == int(host(fl0)[0])
        a2, c = m.resample_permuted("multinomial", w, seed=4, offset=1, filter_base=3)
        assert np.array_equal(host(a2), a) and np.array_equal(host(c), oracle.permute(a)[0])
