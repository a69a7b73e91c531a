"""Metropolis batches with step counts of their own: chunks from the queue,
with more chunks than workgroups and with as many, against equal chunks (no
workspace) and, segment by segment, the oracle."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import _lib, inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def pfr():
    import paper_1301_4019_amd as m
    return m


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("chunk", [1024, 8192])
@pytest.mark.parametrize("kind", ["ragged", "short", "long", "none"])
def test_queue_equals_equal_chunks(dtype, chunk, kind):
    g = np.random.default_rng(chunk + len(kind))
    sizes = {"ragged": np.rint(2.0 ** g.uniform(0, 15, 700)).astype(np.int64),
             "short": g.integers(0, 700, 4096), "long": np.array([300000, 0, 70000, 40000] * 4),
             "none": g.integers(1, 900, 4096)}[kind]
    F = sizes.size
    B = g.integers(-1, 3 if kind == "none" else 50, F).astype(np.int32)
    if kind == "none":
        B[:] = 0
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = inputs.weights(int(off[-1]), 2.0, seed=F, dtype=dtype)
    wd, offd, Bd = (torch.from_numpy(x).cuda() for x in (w, off, B))
    kw = dict(seed=4, offsets=offd, max_len=int(sizes.max()), B_per_filter=Bd)
    need = pfr().workspace_bytes(_lib.OP_METROPOLIS, w.size, offd, int(sizes.max()))
    assert need > 0
    default = pfr().get_tuning()
    pfr().set_tuning(batch_metropolis_chunk=chunk)
    try:
        got = pfr().resample_metropolis(wd, 0, out=torch.full((w.size,), -7, dtype=torch.int32,
                                                              device="cuda"), **kw)
        want = pfr().resample_metropolis(wd, 0, workspace=pfr().new_workspace(256), **kw)
        torch.cuda.synchronize()
    finally:
        pfr().set_tuning(**default)
    assert torch.equal(got, want)
    got = got.cpu().numpy()
    for f in [*range(3), F // 2, F - 1]:
        s = slice(off[f], off[f + 1])
        if sizes[f]:
            assert np.array_equal(got[s], oracle.metropolis_mt(w[s], max(int(B[f]), 0), seed=4,
                                                               filt=f)), f


def test_no_workspace_beyond_4096_segments():
    off = torch.arange(0, 4098, dtype=torch.int64) * 20
    seg = _lib.Segments(4097 * 20, 4097, off.data_ptr(), 20)
    import ctypes
    assert _lib.load().pfr_workspace_bytes(_lib.OP_METROPOLIS, ctypes.byref(seg), 0) == 0
