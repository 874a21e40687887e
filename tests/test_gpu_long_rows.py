"""GPU parity of owners (rows or columns) with many stored pairs: a point far
from the other cloud keeps every point of it (its gap sets its radius). The
softmax kernels and the per-iteration sweeps give such an owner a whole wave
once its pairs exceed the registers of its group of 4 to 16 lanes (8 pairs a
lane); 64 lanes hold 512. Lengths at those edges, against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2512_19743_amd as apml

from .test_gpu_parity import _check_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    apml.load()


def clouds(n, m, far, seed):
    """x: n points of which `far` lie at distance 1 from one point of y and 1.3 to
    1.45 from the other m - 1, so that each of those rows stores all m pairs."""
    rng = np.random.default_rng(seed)
    y = rng.uniform(-0.04, 0.04, (m, 3)) + [1.36, 0.0, 0.0]
    y[0] = [1.0, 0.0, 0.0]
    x = y[rng.integers(1, m, n)] + rng.normal(0.0, 0.004, (n, 3))
    at = rng.choice(n, far, replace=False)
    x[at] = rng.normal(0.0, 1e-3, (far, 3))
    return x.astype(np.float32)[None], y.astype(np.float32)[None]


# pairs of a long row: one below, at and one above 8 per lane of 4, 8 and 16
# lanes, and of a whole wave
@pytest.mark.parametrize("m", [32, 33, 64, 65, 128, 129, 511, 512, 513, 1301])
@pytest.mark.parametrize("swap", [False, True])
def test_long_owners(m, swap):
    X, Y = clouds(300, m, 3, m)
    if swap:
        X, Y = Y, X
    _check_batch(X, Y, f"long {'columns' if swap else 'rows'} of {m}", n_iter=4)


# several long owners in every wave, and all four reverse and softmax variants'
# long loops at once: per-iteration sweeps (more than 64 pieces of 4 pairs)
@pytest.mark.parametrize("far", [1, 40, 300])
def test_many_long_owners(far):
    X, Y = clouds(300, 700, far, far)
    _check_batch(X, Y, f"{far} long rows", n_iter=3)


# waves that look for long owners: more of them where an owner has more than 1024
# pairs; column and row owners at that edge, and short owners only beside them
@pytest.mark.parametrize("m", [1023, 1024, 1025, 1028, 1029])
def test_owners_at_the_full_edge(m):
    X, Y = clouds(1500, m, 2, m)
    _check_batch(X, Y, f"rows of {m}", n_iter=2)
    _check_batch(Y, X, f"columns of {m}", n_iter=2)
