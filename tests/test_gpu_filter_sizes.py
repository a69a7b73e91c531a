"""The filter's move at the edges of its LDS tiers (2048, 16384 and 32768
particles), on lengths that fill no quad, and at extreme observations, against
the oracle's move of the same permuted ancestry."""
import numpy as np
import pytest

import oracle
from test_gpu_filter import PHI, Q, R, check_B, host, pfr, ulp_close

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 2048, 2049, 16384, 16387, 32768, 32769])
def test_move_matches_oracle(n):
    F = 3
    y = np.array([0.3, -1.7])
    flt = pfr().LGSSMFilter(y, F, n, phi=PHI, q=Q, r=R, seed=21, offset=1, filter_base=4)
    flt.reset()
    for t in (1, 2):
        x0, lz0 = host(flt.x), host(flt.log_z)
        flt.step()
        xo, wo, lzo, Bo = oracle.lgssm_move(host(flt.permuted), x0, lz0, F, n, PHI, Q, R, t,
                                            y[t - 1], seed=21, offset=1, filter_base=4)
        # the tolerances of the filter's own test: 2 and 4 units of binary32
        assert ulp_close(host(flt.x), xo, 2)
        assert ulp_close(host(flt.w), wo, 4)
        np.testing.assert_allclose(host(flt.log_z), lzo, rtol=1e-12, atol=1e-12)
        check_B(host(flt.B), Bo, wo, F, n)
        assert int(host(flt.t)[0]) == t + 1
    assert int(host(flt.flags)[0]) == 0


def test_far_observation_underflows_to_zero_weights():
    """Residuals whose exponential underflows give weight 0; the largest is 1."""
    F, n = 2, 1000
    flt = pfr().LGSSMFilter(np.array([1e5]), F, n, phi=PHI, q=Q, r=1e-3, seed=2)
    flt.reset()
    x0, lz0 = host(flt.x), host(flt.log_z)
    flt.step()
    xo, wo, lzo, _ = oracle.lgssm_move(host(flt.permuted), x0, lz0, F, n, PHI, Q, 1e-3, 1, 1e5,
                                       seed=2)
    w = host(flt.w)
    assert ulp_close(host(flt.x), xo, 2)
    assert np.array_equal(w == 0, wo == 0) and np.all(w.reshape(F, n).max(axis=1) == 1.0)
    np.testing.assert_allclose(host(flt.log_z), lzo, rtol=1e-12)


def test_nan_state_stays_nan():
    F, n = 2, 300
    flt = pfr().LGSSMFilter(np.array([0.5]), F, n, phi=PHI, q=Q, r=R, seed=3)
    flt.reset()
    flt.x[7] = float("nan")
    flt.x[n + 299] = float("inf")
    flt.step()
    x, w = host(flt.x), host(flt.w)
    moved = host(flt.permuted)
    assert np.array_equal(np.isnan(x[:n]), moved[:n] == 7)
    assert np.array_equal(np.isnan(w[:n]), moved[:n] == 7)
    assert np.array_equal(np.isinf(x[n:]), moved[n:] == 299) and np.all(w[n:][moved[n:] == 299] == 0)
