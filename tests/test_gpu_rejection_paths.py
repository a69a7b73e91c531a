"""Rejection at the edges of its paths (weights in LDS, bound codes in LDS,
global weights; small and large batches; the tail's lane shares), against the
oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import inputs
from test_gpu_metropolis_long_segments import EDGES, batch
from test_gpu_parity import dev, host, new_flags, pfr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check(w, off, w_max, filter_base=0, max_len=None, **kw):
    """One batched call against the oracle, segment by segment."""
    fl = new_flags()
    per = np.ndim(w_max) > 0
    how = {"w_max_per_filter": dev(np.asarray(w_max, dtype=np.float64))} if per else {}
    a = host(pfr().resample_rejection(dev(w), 1.0 if per else w_max, offsets=dev(off),
                                      max_len=max_len, filter_base=filter_base, flags=fl,
                                      **how, **kw))
    want = 0
    for f in range(len(off) - 1):
        if off[f] < off[f + 1]:
            s = slice(off[f], off[f + 1])
            ref, rfl = oracle.rejection(w[s], w_max[f] if per else w_max, filt=filter_base + f,
                                        **kw)
            assert np.array_equal(a[s], ref), (f, off[f + 1] - off[f])
            want |= rfl
    assert int(host(fl)[0]) & oracle.FLAG_TRIAL_CAP == want & oracle.FLAG_TRIAL_CAP


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_long_segments(dtype):
    ys = [0.0, 4.0, 2.0, 3.0, 1.0, 4.0, 3.5, 2.5, 3.0]
    w, off = batch(EDGES, ys, dtype, 41)
    check(w, off, 1.0, seed=3, offset=2, filter_base=5, max_len=max(EDGES))
    check(w, off, np.linspace(1.0, 2.0, len(EDGES)), seed=4)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("total", [65536, 65537])
def test_small_and_large_batches(dtype, total):
    """Both sides of the 256-particle workgroups' limit, with empty segments,
    segments shorter than a wave, and one that crosses many workgroups; the
    LDS capacity follows max_len."""
    sizes = [0, 1, 63, 64, 0, 65, 2, 4096, 4097, 8192, 16385]
    sizes += [1] * 100 + [total - sum(sizes) - 100, 0]
    g = np.random.default_rng(total)
    w, off = batch(sizes, g.uniform(0, 4, len(sizes)), dtype, total)
    check(w, off, 1.0, seed=8, max_len=max(sizes))
    short = [3000] * (total // 3000) + [total % 3000]
    w, off = batch(short, g.uniform(0, 4, len(short)), dtype, total + 1)
    check(w, off, 1.0, seed=9, max_len=3000)


@pytest.mark.parametrize("n", [1, 2, 3, 5, 31, 33, 63, 64, 65, 100])
@pytest.mark.parametrize("max_trials", [1, 2, 3, 4, 5, 64, 255, 1 << 20])
def test_lane_shares_and_trial_cap(n, max_trials):
    """Few particles at a low acceptance rate: every share of the 64 lanes."""
    sizes = [n] * 7
    w, off = batch(sizes, [4.0] * 7, np.float32, n)
    check(w, off, 4.0, seed=n, max_trials=max_trials)


@pytest.mark.parametrize("dtype,w_max", [(np.float32, 1e39), (np.float32, 1.0),
                                         (np.float64, 1e300), (np.float64, 1.0),
                                         (np.float64, 1e-280), (np.float64, 1e-320),
                                         (np.float32, 0.0)])
@pytest.mark.parametrize("n", [300, 40000])
def test_extreme_weights_and_bounds(dtype, w_max, n):
    """Weights at the ends of the type's range, infinities and NaN, and bounds
    at which products overflow or vanish."""
    g = np.random.default_rng(6)
    info = np.finfo(dtype)
    pool = np.array([0.0, info.smallest_subnormal, info.tiny, info.max, info.max / 2, 1.0, np.inf,
                     np.nan, -1.0, min(w_max, float(info.max))], dtype=dtype)
    w = g.choice(pool, 2 * n)
    off = np.array([0, n, 2 * n], dtype=np.int64)
    check(w, off, [w_max, w_max], seed=2, max_trials=40)
    if w_max > 0:  # a scalar bound of 0 is refused
        check(w, off, w_max, seed=2, max_trials=40)
