"""Batched Metropolis on segments beyond the LDS staging capacity (their bound
codes are staged instead), against the oracle, bit for bit; and the cut of a
batch by cost."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import inputs
from test_gpu_parity import dev, host, pfr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# capacity of the weights (binary32, binary64), of the codes at one, two and
# four particles each, and one past each
EDGES = (16384, 16385, 32768, 32769, 65536, 65537, 131073, 262144, 262145)


def batch(sizes, ys, dtype, seed):
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = np.concatenate([inputs.weights(n, y, seed + i, dtype) if n else np.zeros(0, dtype)
                        for i, (n, y) in enumerate(zip(sizes, ys))])
    return w, off


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_long_segments_bit_exact(dtype):
    ys = [0.0, 4.0, 2.0, 3.0, 1.0, 4.0, 3.5, 2.5, 3.0]
    w, off = batch(EDGES, ys, dtype, 31)
    B = np.array([5, 13, 4, 8, 1, 9, 6, 3, 7], dtype=np.int32)
    for per_filter in (True, False):
        kw = {"B_per_filter": dev(B)} if per_filter else {}
        a = host(pfr().resample_metropolis(dev(w), 6, seed=3, offset=2, filter_base=5,
                                           offsets=dev(off), max_len=max(EDGES), **kw))
        for f in range(len(EDGES)):
            s = slice(off[f], off[f + 1])
            ref = oracle.metropolis(w[s], int(B[f]) if per_filter else 6, seed=3, offset=2,
                                    filt=5 + f)
            assert np.array_equal(a[s], ref), (EDGES[f], per_filter)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [33001, 65536])
def test_single_vector_with_codes(dtype, n):
    w = inputs.weights(n, 3.5, seed=n, dtype=dtype)
    for B in (11, 12, 61):  # plain below 12 steps, codes from there
        a = host(pfr().resample_metropolis(dev(w), B, seed=B))
        assert np.array_equal(a, oracle.metropolis(w, B, seed=B)), B


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_codes_of_extreme_weights(dtype):
    """Zeros, subnormals, the smallest and the largest weights and values on
    both sides of a code's boundary."""
    g = np.random.default_rng(4)
    info = np.finfo(dtype)
    n = 40000
    pool = np.array([0.0, info.smallest_subnormal, 7 * info.smallest_subnormal, info.tiny,
                     info.max, info.max / 2, 1.0, np.nextafter(dtype(1), dtype(2)),
                     np.nextafter(dtype(1), dtype(0)), 1 + 2.0**-7, 1 + 2.0**-4], dtype=dtype)
    w = np.concatenate([g.choice(pool, n // 2),
                        np.ldexp(g.random(n // 2) + 0.5, g.integers(-60, 60, n // 2)).astype(dtype)])
    off = np.array([0, n, 2 * n], dtype=np.int64)
    w2 = np.concatenate([w, g.permutation(w)])
    a = host(pfr().resample_metropolis(dev(w2), 40, seed=9, offsets=dev(off), max_len=n))
    for f in range(2):
        ref = oracle.metropolis(w2[f * n:(f + 1) * n], 40, seed=9, filt=f)
        assert np.array_equal(a[f * n:(f + 1) * n], ref), f


def test_cut_by_cost_covers_every_particle():
    """Step counts from 0 to far above the rest, empty segments, and segments
    shorter than a pass: every particle is resampled, as in single calls."""
    g = np.random.default_rng(12)
    sizes = [0, 70000, 1, 0, 300, 5000, 33000, 0, 1024, 1025, 20000, 0]
    B = np.array([9, 1, 400, 3, 300, 0, 40, 7, 2, 900, 12, 1], dtype=np.int32)
    w, off = batch(sizes, g.uniform(0, 4, len(sizes)), np.float32, 3)
    for max_len in (None, max(sizes)):
        a = host(pfr().resample_metropolis(dev(w), 1, seed=5, B_per_filter=dev(B),
                                           offsets=dev(off), max_len=max_len))
        for f, n in enumerate(sizes):
            if n:
                ref = oracle.metropolis(w[off[f]:off[f + 1]], int(B[f]), seed=5, filt=f)
                assert np.array_equal(a[off[f]:off[f + 1]], ref), (f, max_len)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("segments", [2, 700])
@pytest.mark.parametrize("max_len", ["short", "long", None])
def test_chunks_from_the_queue(dtype, segments, max_len):
    """A batch with its own step counts and a workspace (chunks handed out to
    workgroups that stay) against one without (one workgroup per chunk): every
    LDS tier, more chunks than workgroups, shares that are not whole waves."""
    g = np.random.default_rng(segments)
    top = {"short": 2000, "long": 70000, None: 20000}[max_len]
    sizes = g.integers(0, top if segments == 2 else min(top, 4000), segments)
    sizes[:2] = top, max(1, 66000 - top)  # beyond the small batches' path
    if segments > 2 and max_len == "short":
        sizes[1] = 1999
    B = g.integers(0, 40, segments).astype(np.int32)
    w, off = batch(list(sizes), g.uniform(0, 4, segments), dtype, 5)
    kw = dict(seed=5, offset=1, filter_base=2, B_per_filter=dev(B), offsets=dev(off),
              max_len=None if max_len is None else int(max(sizes)))
    a = [host(pfr().resample_metropolis(dev(w), 1, **kw)) for _ in range(2)]
    b = host(pfr().resample_metropolis(dev(w), 1, workspace=torch.empty(0, dtype=torch.uint8,
                                                                        device="cuda"), **kw))
    assert np.array_equal(a[0], b) and np.array_equal(a[1], b)
    for f in list(range(2)) + [segments - 1]:
        if sizes[f]:
            ref = oracle.metropolis(w[off[f]:off[f + 1]], int(B[f]), seed=5, offset=1, filt=2 + f)
            assert np.array_equal(b[off[f]:off[f + 1]], ref), f
