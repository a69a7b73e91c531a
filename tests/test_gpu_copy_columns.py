"""The copy step on states whose components are not contiguous: even and odd
component counts at the edges of a workgroup's tile, against indexing."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.uint8, torch.float16, torch.float32, torch.float64,
                                   torch.complex128])
@pytest.mark.parametrize("n", [1, 255, 1024, 1025, 3001])
@pytest.mark.parametrize("D", [1, 2, 3, 8, 9])
@pytest.mark.parametrize("pad", [0, 5])
def test_columns(dtype, n, D, pad):
    import paper_1301_4019_amd as pfr
    w = torch.rand(n, generator=torch.Generator().manual_seed(n + D)).cuda()
    _, c = pfr.resample_permuted("multinomial", w, seed=2)
    buf = torch.randint(0, 100, (D + 1, n + pad),
                        generator=torch.Generator().manual_seed(D)).to(dtype).cuda()
    x = buf[:D, pad // 2:pad // 2 + n].t()
    assert tuple(x.shape) == (n, D)
    want = buf.clone()
    want[:D, pad // 2:pad // 2 + n] = x[c.long()].t()
    pfr.copy_particles(c, x)
    assert torch.equal(buf, want)


@pytest.mark.parametrize("n,D,dtype", [(1500001, 17, torch.uint8), (1500001, 3, torch.complex128),
                                       (500009, 13, torch.float64), (48000, 255, torch.float32)])
def test_large_states(n, D, dtype):
    """States on the other side of the rule that copies four particles abreast."""
    import paper_1301_4019_amd as pfr
    w = torch.rand(n, generator=torch.Generator().manual_seed(n)).cuda() ** 4
    _, c = pfr.resample_permuted("systematic", w, seed=2)
    x = torch.randint(0, 100, (D, n), device="cuda").to(dtype).t()
    want = x[c.long()]
    pfr.copy_particles(c, x)
    assert torch.equal(x, want)
