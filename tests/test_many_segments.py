"""Batches of more segments than one launch of 1024-thread workgroups holds."""
import numpy as np
import pytest

import launchlog
from paper_1301_4019_amd import _lib

F = (1 << 22) + 1000


@launchlog.needs_shim
@pytest.mark.parametrize("scheme,max_len", [("stratified", 2000), ("systematic", 10000),
                                            ("systematic", 0)])
def test_launches_stay_within_the_limit(scheme, max_len):
    rc, log = launchlog.run("""
s = ctypes.byref(seg(1 << 28, %d, 5*GB, %d))
result = [lib.resample_%s(16*GB, 0, s, 0, RNG, 32*GB, None, 0, None, None), launches()]
""" % (F, max_len, scheme))
    assert rc == _lib.PFR_OK
    assert all(x[1] * x[2] < 1 << 32 for x in log)
    one = [x for x in log if launchlog.kernel(x) == "k_scan_one" and x[2] == 1024]
    assert one and sum(x[1] for x in one) % F == 0


@pytest.mark.gpu
def test_result():
    """The one-workgroup launches against the block-parallel ones."""
    torch = pytest.importorskip("torch")
    import paper_1301_4019_amd as pfr
    g = np.random.default_rng(5)
    sizes = g.integers(0, 4, F)
    sizes[[0, 77, F - 2, F - 1]] = (1500, 1025, 1200, 3)
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    w = torch.rand(int(off[-1]), generator=torch.Generator(device="cuda").manual_seed(1),
                   device="cuda")
    a = pfr.resample_systematic(w, seed=2, offsets=off, max_len=1500,
                                out=torch.full((w.numel(),), -7, dtype=torch.int32, device="cuda"))
    assert torch.equal(a, pfr.resample_systematic(w, seed=2, offsets=off))
