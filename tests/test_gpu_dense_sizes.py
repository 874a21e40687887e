"""GPU parity of the dense APML path at the edges of its launches: row lengths
around the waves per row of the fused sweep (256, 512, 1024, 2048, 4096, 8192
columns; longer rows take separate row and column products), lengths that are
not a multiple of four, few rows, many iterations (the thin product of the
adjoint in one step of 16 iterations, or several) and scalings that would leave
the range of a double without the powers of two kept out of them."""
import numpy as np
import pytest
import torch

import paper_2512_19743_amd as apml
from oracle.dense import dense_apml
from workloads import custom

from ._parity import GRAD_RTOL, LOSS_RTOL, note, rel_norm
from .test_gpu_dense import _against_oracle, run_dense

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    apml.load()


@pytest.mark.parametrize("N,M", [(3, 2), (5, 3), (65, 63), (64, 256), (67, 257), (130, 512), (33, 514), (70, 1024),
                                 (300, 1025), (64, 2048), (50, 2049), (34, 4096), (35, 4099), (40, 8192), (37, 8195),
                                 (2049, 70), (8200, 20)])
def test_dense_row_lengths(N, M):
    X, Y = custom(65, 2, N, M, reference="sphere", prediction="uniform_cube")
    _against_oracle(X, Y, "sizes", n_iter=3, gbar=[1.0, -0.5])


@pytest.mark.parametrize("L", [2, 15, 16, 17, 33])
def test_dense_thin_product_lengths(L):
    X, Y = custom(66, 3, 90, 150, sigma=0.05)
    _against_oracle(X, Y, f"L={L}", n_iter=L)


# alpha grows by N / M (beta shrinks) in each iteration: 2^(3 * 500) and 2^(-1.6 * 800)
@pytest.mark.parametrize("N,M,L", [(96, 12, 500), (12, 36, 800)])
def test_dense_scalings_stay_in_range(N, M, L):
    X, Y = custom(67, 1, N, M, reference="sphere", prediction="uniform_cube")
    _against_oracle(X, Y, f"range L={L}", n_iter=L)


@pytest.mark.parametrize("d", [1, 3, 4, 7, 8, 9, 16])
def test_dense_dimensions_with_many_points(d):
    rng = np.random.default_rng(200 + d)
    B, N, M = 2, 131, 270
    Y = rng.standard_normal((B, M, d)).astype(np.float32)
    X = (Y[:, rng.permutation(M)[:N]] + 0.2 * rng.standard_normal((B, N, d))).astype(np.float32)
    note(f"dense dimension d={d}")
    loss, gx, gy = run_dense(X, Y, gbar=[1.0, -0.7], n_iter=6)
    for b in range(B):
        x = torch.from_numpy(X[b].astype(np.float64)).requires_grad_(True)
        y = torch.from_numpy(Y[b].astype(np.float64)).requires_grad_(True)
        ref, _ = dense_apml(x, y, tau=0.0, n_iter=6)
        (ref * [1.0, -0.7][b]).backward()
        assert abs(loss[b] - ref.item()) <= LOSS_RTOL * abs(ref.item())
        assert rel_norm(gx[b], x.grad.numpy()) <= GRAD_RTOL
        assert rel_norm(gy[b], y.grad.numpy()) <= GRAD_RTOL


# The kernels' own root and exponential keep a NaN: a sample with a point that
# is not finite shows it in its loss and gradients, and in no other sample's.
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("d", [3, 5])
def test_dense_points_that_are_not_finite(value, d):
    rng = np.random.default_rng(300 + d)
    X, Y = (rng.standard_normal((3, n, d)).astype(np.float32) for n in (70, 130))
    clean = run_dense(X, Y, gbar=[1.0, 1.0, 1.0], n_iter=3)
    for cloud in (X, Y):
        bad = [c.copy() for c in (X, Y)]
        bad[0 if cloud is X else 1][1, 33, d - 1] = value
        note(f"dense {value} in cloud {'X' if cloud is X else 'Y'} d={d}")
        for got, ref in zip(run_dense(*bad, gbar=[1.0, 1.0, 1.0], n_iter=3), clean):
            assert np.isnan(got[1]).all()
            assert np.array_equal(got[0], ref[0]) and np.array_equal(got[2], ref[2])


# A gap clamped to a tiny eps_gap: the temperature times a difference of costs
# passes the range of a double, and the softmax is 1 on the nearest points and 0
# elsewhere, as its limit says.
@pytest.mark.parametrize("eps_gap", [1e-200, 1e-260, 2e-307])
def test_dense_temperature_beyond_range(eps_gap):
    rng = np.random.default_rng(310)
    X, Y = (rng.uniform(-3.0, 3.0, (2, n, 3)).astype(np.float32) for n in (20, 30))
    Y[:, 15:] = Y[:, :15]  # every row's two nearest columns coincide
    loss, gx, gy = run_dense(X, Y, gbar=[1.0, 1.0], n_iter=0, delta=0.0, eps_gap=eps_gap)
    for b in range(2):
        x, y = (torch.from_numpy(c[b].astype(np.float64)) for c in (X, Y))
        D = (x[:, None] - y[None]).square().sum(-1).sqrt()
        P = (D == D.min(1, keepdim=True)[0]).double() * 0.5
        gap = torch.sort(D, 0)[0]
        T = np.log(19 * 0.8 / 0.2) / (gap[1] - gap[0])
        P = 0.5 * (P + torch.softmax(-T * (D - gap[0]), 0))
        ref = (P * D).sum().item()
        assert abs(loss[b] - ref) <= LOSS_RTOL * ref
