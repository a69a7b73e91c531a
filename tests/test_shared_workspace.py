"""One workspace under several host threads: the launches of a call that goes
through a workspace stand together in its stream, whichever threads share the
workspace (a call of another thread in between would overwrite what the first
part left for the second)."""
import numpy as np
import pytest

import launchlog
import oracle
import paper_1301_4019_amd as pfr
from paper_1301_4019_amd import _lib, inputs

CALLS = {
    # (a call on workspace ws, its launches)
    "metropolis_batch": ("lib.resample_metropolis(1*GB, 0, batch, 0, 2*GB, RNG, 3*GB, ws, 1 << 20, None)",
                         2),
    "multinomial_short": ("lib.resample_multinomial(1*GB, 0, short, 0, RNG, 3*GB, ws, 1 << 30, None,"
                          " None)", 2),
    "permuted_metropolis": ("lib.resample_permuted(3, 1*GB, 0, batch, ctypes.byref(params), RNG,"
                            " 3*GB, 4*GB, ws, 1 << 30, None, None)", None),
    "permuted_multinomial": ("lib.resample_permuted(0, 1*GB, 0, short, ctypes.byref(params), RNG,"
                             " 3*GB, 4*GB, ws, 1 << 30, None, None)", None),
    "systematic_long": ("lib.resample_systematic(1*GB, 0, long_, 0, RNG, 3*GB, ws, 1 << 30, None,"
                        " None)", 2),
    "permute_long": ("lib.permute_ancestors(1*GB, long_, 0, 3*GB, ws, 1 << 30, None, None)", 5),
}


@launchlog.needs_shim
@pytest.mark.parametrize("name", sorted(CALLS))
def test_launches_of_a_call_stand_together(name):
    call, count = CALLS[name]
    launches, rcs = launchlog.run("""
batch = ctypes.byref(seg(200000, 100, 5*GB, 5000))
short = ctypes.byref(seg(3000))
long_ = ctypes.byref(seg(100000))
params = _lib.SchemeParams(0, 0, 2*GB, 1.0, None, 1 << 20)
ws, rcs = 8*GB, []
CALL = lambda: rcs.append(%s)
shim.shim_sleep(ctypes.c_long(300000))
CALL()
alone = [x[4] for x in launches()]
ts = [threading.Thread(target=lambda: [CALL() for _ in range(4)]) for _ in range(4)]
for t in ts: t.start()
for t in ts: t.join()
result = [[alone, launches()], rcs]
""" % call)
    alone, together = launches
    assert rcs == [_lib.PFR_OK] * 17
    assert len(alone) == count or (count is None and len(alone) > 1)
    assert len(together) == 16 * len(alone)
    for k in range(0, len(together), len(alone)):
        part = together[k:k + len(alone)]
        assert [x[4] for x in part] == alone and len({x[0] for x in part}) == 1, k


def test_cache_replaces_an_entry_without_counting_it_twice():
    c = pfr._WorkspaceCache(1000)

    class Ws:
        def numel(self):
            return 100
    c.put("k", Ws())
    second = Ws()
    c.put("k", second)  # (two threads that both found nothing)
    assert c.bytes == 100 and c.get("k") is second


# ------------------------------------------------------------------ on the GPU
def _gpu():
    return pytest.importorskip("torch")


def _batch(seed):
    g = np.random.default_rng(seed)
    sizes = g.integers(200, 5000, 60)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    w = np.concatenate([inputs.weights(int(n), 2.0, seed=100 * seed + k)
                        for k, n in enumerate(sizes)])
    B = g.integers(1, 40, 60).astype(np.int32)
    return w, off, B, int(sizes.max())


@pytest.mark.gpu
def test_threads_on_one_stream():
    """Four threads on the default stream, each with its own input: every
    result is the one of a call alone."""
    import threading
    torch = _gpu()
    data = [_batch(k) for k in range(4)]
    short = [inputs.weights(3000, 1.0, seed=50 + k) for k in range(4)]
    dev = [[torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in d[:3]] for d in data]
    sdev = [torch.from_numpy(w).cuda() for w in short]

    def calls(k):
        w, off, B = dev[k]
        kw = dict(seed=k, offsets=off, max_len=data[k][3], B_per_filter=B)
        return (pfr.resample_metropolis(w, 0, **kw), pfr.resample_multinomial(sdev[k], seed=k),
                *pfr.resample_permuted("metropolis", w, **kw),
                *pfr.resample_permuted("multinomial", sdev[k], seed=k))

    want = [calls(k) for k in range(4)]
    torch.cuda.synchronize()
    got = [[] for _ in range(4)]
    ts = [threading.Thread(target=lambda k=k: got[k].extend(calls(k) for _ in range(10)))
          for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for k in range(4):
        assert len(got[k]) == 10
        for r in got[k]:
            assert all(torch.equal(x, y) for x, y in zip(r, want[k])), k
    w, off, B, _ = data[0]
    a = want[0][0].cpu().numpy()
    for f in range(3):
        s = slice(off[f], off[f + 1])
        assert np.array_equal(a[s], oracle.metropolis(w[s], int(B[f]), seed=0, filt=f))
