"""The skipping scans read the clouds in the order of a sort by chunks of 2048
points, merged up to 16 at a time: no point may be lost or doubled at the
chunks' and levels' edges, with equal keys, or where the two clouds have
different numbers of chunks. The stored pairs must be those of the full scan."""
import numpy as np
import pytest
import torch

import paper_2512_19743_amd as apml

from ._parity import note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    apml.load()


def _pairs(x, y, scan):
    loss, plan = apml.apml_forward(x, y, apml.apml_params_default(dense_scan=scan, n_iter=1))
    torch.cuda.synchronize()
    out = [plan.export(b) for b in range(x.shape[0])], plan.info().stored_pairs
    plan.close()
    return out


@pytest.mark.parametrize("B,N,M,cells", [
    (2, 2047, 2049, 0),        # around one chunk
    (1, 4096, 2, 0),           # a cloud of two points
    (1, 64, 6145, 0),          # one and four chunks
    (2, 5000, 12300, 6),       # many equal keys across chunks
    (1, 32768, 32769, 0),      # one level of 16 chunks at most, and two levels
])
def test_merged_sort_keeps_every_point(B, N, M, cells):
    note(f"spatial sort: {B} x {N} x {M} cells={cells}")
    g = np.random.default_rng(N + M)
    X, Y = g.random((B, N, 3), np.float32), g.random((B, M, 3), np.float32)
    if cells:  # clusters far smaller than a cell of the curve
        X = np.floor(X * cells) / cells + 1e-5 * X
        Y = np.floor(Y * cells) / cells + 1e-5 * Y
    x, y = torch.from_numpy(X.astype(np.float32)).cuda(), torch.from_numpy(Y.astype(np.float32)).cuda()
    (full, nf), (skip, ns) = _pairs(x, y, 1), _pairs(x, y, 2)
    assert nf == ns
    for a, b in zip(full, skip):
        for name in ("i", "j", "flags"):
            np.testing.assert_array_equal(a[name], b[name])
