"""Block-parallel batches at the segment counts where the prefix over the
segments changes its workgroup, against calls on the segments alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("F", [2, 255, 256, 257, 1023, 1024, 1025])
@pytest.mark.parametrize("scheme", ["systematic", "multinomial"])
def test_prefix(F, scheme):
    import paper_1301_4019_amd as pfr
    sizes = np.random.default_rng(F).integers(0, 2500, F)
    sizes[[0, F - 1]] = (3000, 1025)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = torch.rand(int(off[-1]), generator=torch.Generator().manual_seed(F)).cuda()
    run = getattr(pfr, "resample_" + scheme)
    offd = torch.from_numpy(off).cuda()
    a = run(w, seed=3, offsets=offd)
    p, c = pfr.resample_permuted(scheme, w, seed=3, offsets=offd)
    assert torch.equal(a, p)
    want = pfr.permute_ancestors(a, sorted_hint=True, offsets=offd)
    assert torch.equal(c, want)
    for f in sorted({0, 1, F // 2, F - 1}):
        if sizes[f]:
            alone = run(w[off[f]:off[f + 1]].clone(), seed=3, filter_base=f)
            assert torch.equal(a[off[f]:off[f + 1]], alone), f
