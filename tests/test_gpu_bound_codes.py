"""Bound codes in LDS, in batches where they pay for their staging (a
workgroup's particles times the steps or trials of each reach the segment's
length), at the edges of one, two and four weights a code, on weights of every
kind; and workgroups on both sides of that rule in one call.  Against the
oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import inputs
from test_gpu_metropolis_long_segments import batch
from test_gpu_parity import dev, host, pfr
from test_gpu_rejection_paths import check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

EDGES = (16385, 32769, 65535, 65536, 65537, 131071, 131074, 262143, 262144, 262145)


def metropolis(w, off, B, which, **kw):
    a = host(pfr().resample_metropolis(dev(w), 0, B_per_filter=dev(B), seed=3, offsets=dev(off),
                                       **kw))
    a2 = host(pfr().resample_metropolis(dev(w), 0, B_per_filter=dev(B), seed=3, offsets=dev(off),
                                        workspace=pfr().new_workspace(256), **kw))
    assert np.array_equal(a, a2)
    for f in which:
        s = slice(off[f], off[f + 1])
        assert np.array_equal(a[s], oracle.metropolis_mt(w[s], int(B[f]), seed=3, filt=f)), f


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", EDGES)
def test_edges(dtype, n):
    # more than 2^18 particles: chunks of more than one pass
    sizes = [n, 5, n] + [20000] * 14
    w, off = batch(sizes, [2.0, 1.0, 3.5] + [1.0] * 14, dtype, n)
    B = np.array([90, 3, 130] + [2] * 14, dtype=np.int32)
    metropolis(w, off, B, (0, 1, 2, 5), max_len=max(sizes))
    # 1 % acceptance and lower: a hundred trials and more a particle
    check(w, off, [1.0, 1.0, 30.0] + [1.0] * 14, seed=4, max_trials=300, max_len=max(sizes))


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_extreme_weights(dtype):
    g = np.random.default_rng(4)
    info = np.finfo(dtype)
    n, F = 40000, 8
    pool = np.array([0.0, -0.0, info.smallest_subnormal, 7 * info.smallest_subnormal, info.tiny,
                     info.max, info.max / 2, 1.0, np.nextafter(dtype(1), dtype(2)),
                     np.nextafter(dtype(1), dtype(0)), 1 + 2.0**-7, 1 + 2.0**-4], dtype=dtype)
    w = np.concatenate([np.concatenate([g.choice(pool, n // 2), np.ldexp(
        g.random(n // 2) + 0.5, g.integers(-60, 60, n // 2)).astype(dtype)]) for _ in range(F)])
    bad = g.choice(w.size, 200, replace=False)
    off = np.arange(F + 1, dtype=np.int64) * n
    metropolis(w, off, np.full(F, 40, np.int32), range(F), max_len=n)
    # invalid weights have no defined ancestry: that of chains without codes (a
    # call on the segment alone)
    w[bad] = g.choice(np.array([np.inf, np.nan, -1.0, -np.inf], dtype=dtype), bad.size)
    metropolis(w, off, np.full(F, 40, np.int32), (), max_len=n)
    a = host(pfr().resample_metropolis(dev(w), 40, seed=3, offsets=dev(off), max_len=n))
    for f in range(F):
        s = slice(off[f], off[f + 1])
        alone = host(pfr().resample_metropolis(dev(w[s]), 40, seed=3, filter_base=f))
        assert np.array_equal(a[s], alone), f
    for w_max in (1.0, 2.0**127, 2.0**128, 1e-300):
        check(w, off, [w_max] * F, seed=2, max_trials=60, max_len=n)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [40001, 65537, 200000])
def test_both_sides_of_the_rule(dtype, n):
    """Segments of one length with 0 .. 200 steps, 0.1 to 70 % acceptance."""
    F = 12
    w, off = batch([n] * F, np.linspace(0, 4, F), dtype, n)
    B = np.array([0, 1, 2, 5, 8, 12, 16, 24, 40, 80, 120, 200], dtype=np.int32)
    metropolis(w, off, B, range(F), max_len=n)
    check(w, off, np.linspace(1.0, 20.0, F), seed=6, max_trials=100, max_len=n)
