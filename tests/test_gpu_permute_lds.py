"""Permutation of batches in LDS: segment lengths at the edges of the three
tiers, of the claim window and of a wave, against the oracle's Code 10."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import dev, host, new_flags, pfr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = (1, 64, 65, 2047, 2048, 2049, 16384, 16385, 32768, 32769, 65535, 65536, 65537)
# segments beyond 16384 are permuted in LDS when the batch holds 2^21 particles
COPIES = (1, 8)


def ancestry(kind, n, g):
    if kind == "identity":
        return np.arange(n)
    if kind == "one parent":
        return np.full(n, n // 2)
    if kind == "long chain":  # 0 0 1 2 ...: a walk through many slots
        a = np.arange(n)
        a[max(0, n - 1000):] -= 1
        return np.maximum(a, 0)
    p = g.random(n) ** 6
    return g.choice(n, size=n, p=p / p.sum())


@pytest.mark.parametrize("hint", [True, False])
@pytest.mark.parametrize("with_max_len", [True, False])
@pytest.mark.parametrize("kind", ["random", "identity", "one parent", "long chain"])
@pytest.mark.parametrize("copies", COPIES)
def test_batch_tiers_match_code_10(kind, hint, with_max_len, copies):
    g = np.random.default_rng(len(kind) + 2 * hint)
    sizes = SIZES * copies
    parts = [ancestry(kind, n, g).astype(np.int32) for n in sizes]
    if hint:
        parts = [np.sort(p) for p in parts]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    assert (off[-1] >= 1 << 21) == (copies > 1)
    fl = new_flags()
    c = host(pfr().permute_ancestors(dev(np.concatenate(parts)), sorted_hint=hint,
                                     offsets=dev(off),
                                     max_len=max(SIZES) if with_max_len else None, flags=fl))
    for f, p in enumerate(parts):
        assert np.array_equal(c[off[f]:off[f + 1]], oracle.permute(p)[0]), sizes[f]
    assert int(host(fl)[0]) == 0


@pytest.mark.parametrize("hint", [True, False])
@pytest.mark.parametrize("copies", COPIES)
def test_batch_tiers_out_of_range_ancestors(hint, copies):
    """Values outside a segment count as their own index and raise the flag."""
    g = np.random.default_rng(5)
    sizes = [n for n in SIZES if 2 < n <= 65536] * copies
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    parts = []
    for n in sizes:
        p = np.sort(ancestry("random", n, g)).astype(np.int32)
        p[[0, n - 1]] = [-2**31, 2**31 - 1]  # as their own index: still sorted
        if not hint:
            p[[1, n // 2]] = [-1, n]
        parts.append(p)
    fl = new_flags()
    c = host(pfr().permute_ancestors(dev(np.concatenate(parts)), sorted_hint=hint,
                                     offsets=dev(off), max_len=65536, flags=fl))
    for f, p in enumerate(parts):
        assert np.array_equal(c[off[f]:off[f + 1]], oracle.permute(p)[0]), sizes[f]
    assert int(host(fl)[0]) == pfr().FLAG_BAD_ANCESTOR


def test_batch_equal_segments_skip_the_shorter_tiers():
    """Every segment of the stated length: one tier runs."""
    g = np.random.default_rng(6)
    for n, filters in ((100, 700), (5000, 600), (20000, 300), (40000, 260)):
        parts = [np.sort(ancestry("random", n, g)).astype(np.int32) for _ in range(3)]
        a = np.concatenate([parts[f % 3] for f in range(filters)])
        off = np.arange(filters + 1, dtype=np.int64) * n
        c = host(pfr().permute_ancestors(dev(a), sorted_hint=True, offsets=dev(off), max_len=n))
        ref = [oracle.permute(p)[0] for p in parts]
        for f in range(filters):
            assert np.array_equal(c[off[f]:off[f + 1]], ref[f % 3]), (n, f)


def test_unsorted_input_is_found_out_in_lds():
    """A sorted hint is verified where the segment is permuted in LDS."""
    g = np.random.default_rng(8)
    for n, filters in ((64, 10), (3000, 700), (30000, 300), (60000, 260)):
        p = ancestry("random", n, g).astype(np.int32)
        c = host(pfr().permute_ancestors(dev(np.tile(p, filters)), sorted_hint=True,
                                         offsets=dev(np.arange(filters + 1, dtype=np.int64) * n),
                                         max_len=n))
        assert np.array_equal(c, np.tile(oracle.permute(p)[0], filters)), n
