"""Metropolis chains that gather from global memory: one vector too long for
LDS, few steps, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [32769, 65537, 70001])
@pytest.mark.parametrize("B", [0, 1, 4, 5, 11])
def test_matches_oracle(dtype, n, B):
    import paper_1301_4019_amd as pfr
    w = inputs.weights(n, 2.0, seed=n + B, dtype=dtype)
    wd = torch.from_numpy(w).cuda()
    want = oracle.metropolis_mt(w, B, seed=5, filt=3, offset=2)
    kw = dict(seed=5, filter_base=3, offset=2)
    assert np.array_equal(pfr.resample_metropolis(wd, B, **kw).cpu().numpy(), want)
    Bd = torch.tensor([B], dtype=torch.int32, device="cuda")
    assert np.array_equal(pfr.resample_metropolis(wd, 99, B_per_filter=Bd, **kw).cpu().numpy(),
                          want)
