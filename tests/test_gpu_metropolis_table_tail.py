"""Metropolis through the bound table where a workgroup's chunk leaves a
remainder of one, two or more chains a lane after its full passes, against the
oracle."""
import numpy as np
import pytest

import oracle
from paper_1301_4019_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# particles of a workgroup: 256 of them share the vector
@pytest.mark.parametrize("dtype,chunks", [(np.float32, [4097, 5120, 5121, 6144, 6145]),
                                          (np.float64, [2049, 3072, 3073])])
def test_remainder(dtype, chunks):
    import paper_1301_4019_amd as pfr
    for chunk in chunks:
        n = 256 * chunk - 3
        w = inputs.weights(n, 2.0, seed=chunk, dtype=dtype)
        a = pfr.resample_metropolis(torch.from_numpy(w).cuda(), 61, seed=5).cpu().numpy()
        assert np.array_equal(a, oracle.metropolis_mt(w, 61, seed=5)), chunk


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("n", [65535, 65536, 65537])
def test_shortest(n, dtype):
    """Both sides of the length from which the table is used."""
    import paper_1301_4019_amd as pfr
    w = inputs.weights(n, 2.0, seed=n, dtype=dtype)
    a = pfr.resample_metropolis(torch.from_numpy(w).cuda(), 61, seed=5).cpu().numpy()
    assert np.array_equal(a, oracle.metropolis_mt(w, 61, seed=5))
