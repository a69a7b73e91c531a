"""Row copies in pieces of 1 to 16 bytes: row lengths, strides and addresses
that allow each width, rows of one, a few and many pieces, padded rows; and
the counts of Code 12 at the edges of its tiles of values."""
import numpy as np
import pytest

import oracle
from test_gpu_aux_exports import permuted_ancestry
from test_gpu_parity import dev, host, pfr

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 255, 1025, 3001])
@pytest.mark.parametrize("elem", [torch.uint8, torch.int16, torch.float32, torch.float64])
def test_rows_of_every_width(n, elem):
    c = permuted_ancestry(n, np.random.default_rng(n)) if n > 1 else np.zeros(1, np.int32)
    for dim, pitch, first in ((1, 1, 0), (2, 2, 0), (3, 3, 0), (4, 4, 0), (4, 5, 0), (4, 4, 1),
                              (8, 8, 0), (12, 16, 4), (16, 16, 0), (16, 17, 0), (17, 17, 0),
                              (64, 64, 0), (67, 70, 3), (300, 300, 0)):
        flat = (torch.arange(first + n * pitch, device="cuda") * 7 % 251).to(elem)
        x = flat[first:].reshape(n, pitch)[:, :dim]
        ref = host(flat).copy()
        rows = ref[first:].reshape(n, pitch)
        rows[:, :dim] = rows[c][:, :dim]
        pfr().copy_particles(dev(c), x)
        assert np.array_equal(host(flat), ref), (dim, pitch, first)  # padding untouched


@pytest.mark.parametrize("n", [1023, 1024, 1025, 100003])
def test_sorted_counts_at_tile_edges(n):
    g = np.random.default_rng(n)
    for a in (np.arange(n), np.zeros(n), np.full(n, n - 1), np.sort(g.integers(0, n, n)),
              np.sort(g.integers(0, 5, n) * (n // 5))):
        o = host(pfr().ancestors_to_offspring(dev(a.astype(np.int32)), sorted_hint=True))
        assert np.array_equal(o, np.bincount(a.astype(np.int64), minlength=n))
