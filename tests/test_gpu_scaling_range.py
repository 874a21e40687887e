"""Clouds of different lengths under many iterations: the unit marginals cannot
both hold, so alpha grows and beta shrinks by about N / M in every iteration.
The reverse sweeps multiply by the squares of the scalings, which pass the
range of a double long before the scalings themselves do. Gradients against
the CPU oracle where one side's scalings reach 1e170 to 1e215, in the register
kernels (clouds up to 2048 points), the streamed ones (up to 8192) and the
per-iteration launches (an owner of more than 256 pairs)."""
import numpy as np
import pytest
import torch

import paper_2512_19743_amd as apml
from workloads import custom

from .test_gpu_parity import _check_batch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    apml.load()


@pytest.mark.parametrize("N,M,L,tau", [
    (200, 12, 175, 0.0),     # registers: 200 pairs a column at most
    (2100, 150, 150, 1e-8),  # streamed
    (400, 10, 120, 0.0),     # per iteration: 400 pairs a column
])
@pytest.mark.parametrize("swap", [False, True])
def test_gradients_where_squared_scalings_overflow(N, M, L, tau, swap):
    X, Y = custom(68, 1, N, M, reference="sphere", prediction="uniform_cube")
    if swap:
        X, Y = Y, X
    _, res = _check_batch(X, Y, f"scalings' range L={L}", n_iter=L, tau=tau)
    assert all(np.isfinite([r["gx_rel"], r["gy_rel"]]).all() for r in res)
