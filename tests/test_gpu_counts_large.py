"""Counts of a sorted ancestry on both sides of the length from which a vector
goes in larger tiles, against torch's bincount."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3 << 21, (3 << 21) + 1, (1 << 23) + 4095])
def test_sorted_counts(n):
    import paper_1301_4019_amd as pfr
    g = torch.Generator(device="cuda").manual_seed(n)
    for power in (1.0, 4.0):
        a = (n * torch.rand(n, generator=g, device="cuda", dtype=torch.float64) ** power)
        a = a.to(torch.int32).sort().values
        o = pfr.ancestors_to_offspring(a, sorted_hint=True)
        assert torch.equal(o.long(), torch.bincount(a.long(), minlength=n))
