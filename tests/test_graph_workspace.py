"""Workspaces under graph capture: a call that is captured gets a workspace of
its graph, not the cached one of the stream it is captured on.  torch captures
every graph on one stream by default, and two such graphs may be replayed at
the same time."""
import pytest

import paper_1301_4019_amd as pfr
from paper_1301_4019_amd import _lib, inputs


class FakeTorch:
    """torch as far as the workspace cache uses it."""
    uint8 = "uint8"

    def __init__(self):
        self.capturing = False
        self._C = self

    def _cuda_isCurrentStreamCapturing(self):
        return self.capturing

    def empty(self, nbytes, dtype=None, device=None):
        class Ws:
            def numel(self):
                return nbytes

            def data_ptr(self):
                return 4096
        return Ws()


def test_captured_calls_get_their_own_workspace(monkeypatch):
    torch = FakeTorch()
    zeroed = []
    monkeypatch.setattr(pfr, "_torch", lambda: torch)
    monkeypatch.setattr(pfr, "_stream", lambda: 7)
    monkeypatch.setattr(pfr, "_WS_CACHE", pfr._WorkspaceCache(1 << 30))
    monkeypatch.setattr(pfr, "_zero_workspace", lambda ws, nbytes: zeroed.append(nbytes))
    seg = _lib.Segments(1 << 17, 1, None, 1 << 17)

    def ws(op):
        return pfr._workspace(op, seg, 0, "cuda:0", None, 7)[0]

    eager = ws(_lib.OP_SYSTEMATIC)
    assert ws(_lib.OP_SYSTEMATIC) is eager and len(zeroed) == 1
    torch.capturing = True
    first, second = ws(_lib.OP_SYSTEMATIC), ws(_lib.OP_SYSTEMATIC)
    assert len({id(eager), id(first), id(second)}) == 3
    # only the expansion of offspring counts needs zeros to start from
    assert len(zeroed) == 1
    assert ws(_lib.OP_OFFSPRING_TO_ANCESTORS) is not None and len(zeroed) == 2
    torch.capturing = False
    assert ws(_lib.OP_SYSTEMATIC) is eager


@pytest.mark.gpu
def test_default_stream_cannot_be_captured():
    """What lets a call on it go without asking."""
    torch = pytest.importorskip("torch")
    torch.zeros(1, device="cuda")
    assert pfr._stream() == 0 and torch.cuda.default_stream().cuda_stream == 0
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        inside = pfr._stream()
        torch.zeros(1, device="cuda")
    assert inside != 0


@pytest.mark.gpu
def test_graphs_replayed_on_two_streams():
    torch = pytest.importorskip("torch")
    n = 300000
    w = [torch.from_numpy(inputs.weights(n, y, seed=9)).cuda() for y in (1.0, 3.0)]
    o = [torch.bincount(pfr.resample_systematic(x, seed=1).long(), minlength=n).int() for x in w]

    def calls(k):
        a, c = pfr.resample_permuted("multinomial", w[k], seed=k)
        return a, c, pfr.offspring_to_ancestors(o[k]), pfr.resample_multinomial(w[k][:2000], seed=k)

    want = [calls(k) for k in range(2)]
    torch.cuda.synchronize()
    graphs, outs = [], []
    for k in range(2):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            outs.append(calls(k))
        graphs.append(g)
    streams = [torch.cuda.Stream() for _ in range(2)]
    for _ in range(20):
        for k in range(2):
            with torch.cuda.stream(streams[k]):
                graphs[k].replay()
    torch.cuda.synchronize()
    for k in range(2):
        assert all(torch.equal(x, y) for x, y in zip(outs[k], want[k])), k
