"""The permutation of batches with segments longer than the stated max_len, at
every tier that can end such a call: the oracle's permutation, as without one."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import _lib

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def pfr():
    import paper_1301_4019_amd as m
    return m


# (the stated longest segment, the segments' lengths); the last three have the
# particles from which segments beyond 16384 are permuted in LDS too
CASES = [(300, [300, 2049, 2048, 70000]), (2048, [2048] * 300 + [2050]),
         (4000, [17, 4000, 16384, 16385]), (16384, [64] * 600 + [20000, 16384]),
         (20000, [20000, 100, 33000] + [2048] * 1024), (32768, [32768, 70000] + [2048] * 1024),
         (65536, [65536, 65537, 1] + [2048] * 1024)]


@pytest.mark.parametrize("max_len,sizes", CASES)
@pytest.mark.parametrize("kind", ["sorted", "unsorted", "invalid"])
@pytest.mark.parametrize("noalloc", [False, True])
def test_permutation(max_len, sizes, kind, noalloc):
    g = np.random.default_rng(max_len)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    parts = [(g.random(n) ** 3 * n).astype(np.int32) for n in sizes]
    if kind == "sorted":
        parts = [np.sort(p) for p in parts]
    if kind == "invalid":
        for p in parts:
            p[len(p) // 2] = -1
            p[-1] = len(p)
    a = torch.from_numpy(np.concatenate(parts)).cuda()
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.full_like(a, -7)
    fn = pfr().permute_ancestors_noalloc if noalloc else pfr().permute_ancestors
    fn(a, sorted_hint=kind == "sorted", offsets=torch.from_numpy(off).cuda(), max_len=max_len,
       out=out, flags=flags)
    torch.cuda.synchronize()
    c = out.cpu().numpy()
    for f, p in enumerate(parts):
        clean = np.where((p < 0) | (p >= len(p)), np.arange(len(p)), p).astype(np.int32)
        assert np.array_equal(c[off[f]:off[f + 1]], oracle.permute(clean)[0]), (f, len(p))
    assert int(flags.cpu()[0]) == (_lib.FLAG_BAD_ANCESTOR if kind == "invalid" else 0)
