"""Batches of the strata schemes that state their longest segment (at most
16384): one workgroup per segment or block-parallel, by how full the
workgroups would be, with the same results."""
import numpy as np
import pytest

import launchlog
from paper_1301_4019_amd import _lib

# (scheme, segments, longest, particles, block-parallel)
CASES = [("systematic", 4096, 1024, 1 << 20, False), ("systematic", 256, 16384, 1 << 20, False),
         ("systematic", 1 << 14, 1100, 1 << 24, True), ("stratified", 1 << 14, 1100, 1 << 24, False),
         ("systematic", 1 << 14, 4096, 9 << 20, False), ("systematic", 8192, 4096, 9 << 20, True),
         ("systematic", 8192, 4096, 22 << 20, False), ("systematic", 8192, 4096, 15 << 20, False),
         ("systematic", 8192, 2048, 1 << 24, True), ("systematic", 4096, 4096, 9 << 19, False),
         ("systematic", 4096, 4096, (9 << 19) + 1, True),
         ("stratified", 300, 4097, 300 * 4097, False), ("stratified", 300, 4097, 3 << 18, False),
         ("stratified", 300, 4097, (3 << 18) + 1, True), ("stratified", 2000, 5000, 10**7, True),
         ("stratified", 1280, 6600, 1280 * 6600, False), ("stratified", 1024, 16384, 1 << 24, False)]


@launchlog.needs_shim
def test_route():
    """With the workspace reported for it; one that is too small, misaligned or
    over one of the call's arrays, or none, leaves one workgroup per segment."""
    got = launchlog.run("""
result = []
for scheme, F, m, n, _ in %s:
    s = ctypes.byref(seg(n, F, 5*GB, m))
    op = getattr(_lib, "OP_" + scheme.upper())
    need = lib.pfr_workspace_bytes(op, s, 0)
    for ws, size in ((64*GB, need), (64*GB, need - 1), (64*GB + 8, need), (16*GB, need),
                     (5*GB, need), (None, 0)):
        rc = getattr(lib, "resample_" + scheme)(16*GB, 0, s, 0, RNG, 32*GB, ws, size, None, None)
        result.append([rc, launches()])
""" % (CASES,))
    for k, (scheme, F, m, n, blocks) in enumerate(CASES):
        for j in range(6):
            rc, log = got[6 * k + j]
            assert rc == _lib.PFR_OK, (CASES[k], j)
            one = [launchlog.kernel(x) == "k_scan_one" for x in log]
            assert one and all(x != (blocks and j == 0) for x in one), (CASES[k], j, log)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("scheme,sizes", [("stratified", [4097] + [2650] * 299),
                                          ("systematic", [1025] + [801] * 5999 + [0, 5])])
def test_result(scheme, sizes, dtype):
    torch = pytest.importorskip("torch")
    import paper_1301_4019_amd as pfr
    off = torch.from_numpy(np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)).cuda()
    w = torch.from_numpy(np.random.default_rng(3).random(sum(sizes)).astype(dtype)).cuda()
    run = getattr(pfr, "resample_" + scheme)
    kw = dict(seed=4, offsets=off, max_len=max(sizes))
    fresh = lambda: torch.full((w.numel(),), -7, dtype=torch.int32, device="cuda")
    a = run(w, out=fresh(), **kw)
    small = torch.zeros(256, dtype=torch.uint8, device="cuda")
    assert torch.equal(a, run(w, out=fresh(), workspace=small, **kw))
    p, c = pfr.resample_permuted(scheme, w, **kw)
    assert torch.equal(a, p)
