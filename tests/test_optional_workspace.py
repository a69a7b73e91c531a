"""A workspace that a call can do without and that lies over one of the call's
arrays is not written to: the call runs without it (Metropolis batches with
step counts of their own, short multinomial vectors).  On the recorded
launches, without a GPU."""
import pytest

import launchlog
from paper_1301_4019_amd import _lib

F, N = 100, 200000  # the batch: segments, particles; its workspace: 1 KB + 1 KB
SETUP = """
F, N = %d, %d
need = lib.pfr_workspace_bytes(_lib.OP_METROPOLIS, ctypes.byref(seg(N, F, 5*GB, 5000)), 0)
perm = lib.pfr_workspace_bytes(_lib.OP_PERMUTE, ctypes.byref(seg(N, F, 5*GB, 5000)), 0)
w, B, a, c, off, t, ws = 1*GB, 2*GB, 3*GB, 4*GB, 5*GB, 6*GB, 8*GB
flags = 9*GB
""" % (F, N)


def metropolis(change, permuted=False):
    call = ("lib.resample_permuted(3, w, 0, s, ctypes.byref(_lib.SchemeParams(0, 0, B, 1.0, None, 9)),"
            " rng, a, c, ws, perm + need, None, None)" if permuted else
            "lib.resample_metropolis(w, 0, s, 0, B, rng, a, ws, need, None)")
    rc, log = launchlog.run(SETUP + change + """
s = ctypes.byref(seg(N, F, off, 5000))
rng = _lib.Rng(1, 0, 0, t)
result = [%s, launches()]
""" % call)
    assert rc == _lib.PFR_OK
    return [launchlog.kernel(x) for x in log]


@launchlog.needs_shim
@pytest.mark.parametrize("array", ["w = ws + need - 4", "w = ws - 4 * N + 4", "a = ws + need - 256",
                                   "a = ws", "B = ws + 1024", "B = ws - 4 * F + 4",
                                   "off = ws + need - 8", "t = ws + 128"])
def test_metropolis_batch(array):
    assert metropolis("") == ["k_cost_prefix", "k_metropolis_staged"]
    assert metropolis(array) == ["k_metropolis_staged"]


@launchlog.needs_shim
@pytest.mark.parametrize("array", ["B = ws + perm + 1024", "off = ws + perm", "t = ws + perm + 128",
                                   "w = ws + perm + need - 4"])
def test_permuted_metropolis_batch(array):
    plain = metropolis("", permuted=True)
    assert plain[:2] == ["k_cost_prefix", "k_metropolis_staged"]
    assert metropolis(array, permuted=True) == plain[1:]


@launchlog.needs_shim
@pytest.mark.parametrize("array", ["t = ws + 64", "flags = ws + 512", "w = ws + 4096", "a = ws - 4"])
def test_short_multinomial(array):
    def kernels(change):
        rc, log = launchlog.run(SETUP + change + """
rng = _lib.Rng(1, 0, 0, t)
result = [lib.resample_multinomial(w, 0, ctypes.byref(seg(3000)), 0, rng, a, ws, 1 << 20, flags,
                                   None), launches()]
""")
        assert rc == _lib.PFR_OK
        return [launchlog.kernel(x) for x in log]
    assert kernels("") == ["k_scan_records_w", "k_scan_emit_mb"]
    assert kernels(array) == ["k_scan_batched"]
