"""Batches with segments longer than the LDS permutation takes: those that go
to the global kernels whole and those of which the shorter segments stay in
LDS, on both sides of each line, against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [66000] * 10 + [30000] * 60,                # 2.4 M particles, 35 K on average
    [70000] * 20 + [40000] * 65,                # 4 M, 47 K
    [90000] * 20 + [53000] * 50,                # 4.4 M, 63 K
    [150000] * 10 + [70000] * 10,               # 2.2 M, 110 K: all longer
    [65536] * 15 + [65537] * 15 + [300] * 3 + [20000] * 20])
@pytest.mark.parametrize("is_sorted", [True, False])
@pytest.mark.parametrize("known", [True, False])
def test_permutation(sizes, is_sorted, known):
    import paper_1301_4019_amd as pfr
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    g = np.random.default_rng(len(sizes))
    a = np.concatenate([(n * g.random(n) ** 3).astype(np.int32) for n in sizes])
    if is_sorted:
        for k in range(len(sizes)):
            a[off[k]:off[k + 1]].sort()
    offd = torch.from_numpy(off).cuda()
    c = pfr.permute_ancestors(torch.from_numpy(a).cuda(), sorted_hint=is_sorted, offsets=offd,
                              max_len=max(sizes) if known else None).cpu().numpy()
    for k in range(0, len(sizes), 7):
        s = slice(off[k], off[k + 1])
        assert np.array_equal(c[s], oracle.permute(a[s])[0]), k
    same = np.concatenate([np.sort(a[off[k]:off[k + 1]]) for k in range(len(sizes))])
    assert np.array_equal(np.concatenate([np.sort(c[off[k]:off[k + 1]])
                                          for k in range(len(sizes))]), same)
