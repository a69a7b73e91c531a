"""Batches with a segment longer than the stated max_len: no output is left
unwritten.  The collective schemes give such a segment its ancestry or the
identity with a flag (in both outputs, when the permutation comes with it),
and every other segment its own result."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import _lib, inputs
from test_gpu_parity import check_collective

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def pfr():
    import paper_1301_4019_amd as m
    return m


def batch(sizes, dtype=np.float32):
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = np.concatenate([inputs.weights(n, 2.0, seed=n + k, dtype=dtype)
                        for k, n in enumerate(sizes)])
    return w, off


# (the stated longest segment, the segments' lengths): one tier each, and many
# short segments, whose tiers are launches of their own
CASES = [(1000, [700, 1500, 1000]), (1024, [1024, 1025, 5, 20000]),
         (3000, [3000, 4097, 17, 2048]), (16384, [16384, 16385, 300, 30000]),
         (900, [900] * 299 + [1100]), (4000, [64] * 300 + [4500, 4000])]


@pytest.mark.parametrize("scheme", ["stratified", "systematic"])
@pytest.mark.parametrize("max_len,sizes", CASES)
@pytest.mark.parametrize("permuted", [False, True])
def test_collective(scheme, max_len, sizes, permuted):
    w, off = batch(sizes)
    wd, offd = torch.from_numpy(w).cuda(), torch.from_numpy(off).cuda()
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    a = torch.full((w.size,), -7, dtype=torch.int32, device="cuda")
    c = torch.full_like(a, -7)
    kw = dict(seed=3, offsets=offd, max_len=max_len, out=a, flags=flags)
    if permuted:
        pfr().resample_permuted(scheme, wd, permuted=c, **kw)
    else:
        getattr(pfr(), "resample_" + scheme)(wd, **kw)
    torch.cuda.synchronize()
    a, c = a.cpu().numpy(), c.cpu().numpy()
    identity = 0
    for f, n in enumerate(sizes):
        s = slice(off[f], off[f + 1])
        if n > max_len and np.array_equal(a[s], np.arange(n)):
            identity += 1
            assert not permuted or np.array_equal(c[s], np.arange(n)), f
            continue
        check_collective(scheme, w[s], a[s], seed=3, filt=f)
        if permuted:
            assert np.array_equal(c[s], oracle.permute(a[s])[0]), f
    assert int(flags.cpu()[0]) == (_lib.FLAG_BAD_COUNTS if identity else 0)
