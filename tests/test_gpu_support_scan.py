"""The full support scan finds candidates on the matrix cores (products of
bfloat16 parts, with the error taken off the thresholds) and tests every hit
again exactly: it must store the pairs of the skipping scan, which evaluates
the exact test alone, for clouds whose scale, offset and thresholds strain the
products: far from the origin, tiny, huge (beyond the products' range, where
the exact scan runs), duplicated points, infinite thresholds, and sizes at the
edges of its tiles (32 x 32 pairs, 64 rows a wave, 128 staged columns)."""
import numpy as np
import pytest
import torch

import paper_2512_19743_amd as apml
from workloads import custom

from ._parity import note

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    apml.load()


def _pairs(X, Y, scan, **prm):
    x, y = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    loss, plan = apml.apml_forward(x, y, apml.apml_params_default(dense_scan=scan, n_iter=2, **prm))
    torch.cuda.synchronize()
    out = [plan.export(b) for b in range(X.shape[0])], plan.info().stored_pairs, loss.cpu().numpy()
    plan.close()
    return out


def _same(X, Y, label, **prm):
    note(f"support scan {label}: {X.shape[0]} x {X.shape[1]} x {Y.shape[1]}")
    X, Y = np.ascontiguousarray(X, np.float32), np.ascontiguousarray(Y, np.float32)
    full, nf, lf = _pairs(X, Y, 1, **prm)
    skip, ns, ls = _pairs(X, Y, 2, **prm)
    assert nf == ns
    for f, s in zip(full, skip):
        assert np.array_equal(f["i"], s["i"]) and np.array_equal(f["j"], s["j"])
        assert np.array_equal(f["flags"], s["flags"])
    assert np.allclose(lf, ls, rtol=1e-6)


@pytest.mark.parametrize("N,M", [(2, 2), (31, 33), (63, 65), (64, 128), (65, 129), (255, 257), (256, 256),
                                 (257, 511), (300, 1000), (1025, 700)])
def test_tile_edges(N, M):
    X, Y = custom(96, 2, N, M, reference="primitives", prediction="perm_noise", sigma=0.05)
    _same(X, Y, "edges")


@pytest.mark.parametrize("scale", [1e-17, 1e-10, 1e-3, 1e3, 1e9, 1e14, 1e16])
def test_scales(scale):
    X, Y = custom(97, 2, 300, 400, sigma=0.05)
    _same(X * np.float32(scale), Y * np.float32(scale), f"scale {scale}", eps_gap=1e-6 * scale, delta=1e-8 * scale)


@pytest.mark.parametrize("offset", [1.0, 30.0, 1000.0])
def test_far_from_the_origin(offset):
    X, Y = custom(98, 2, 500, 450, sigma=0.05)
    _same(X + np.float32(offset), Y + np.float32(offset), f"offset {offset}")


def test_one_point_out_of_range():
    # the exact scan takes the tiles that hold it
    X, Y = custom(99, 1, 600, 900, sigma=0.05)
    X[0, 300] = [3e16, 0.0, 0.0]
    _same(X, Y, "far row")
    X, Y = custom(99, 1, 600, 900, sigma=0.05)
    Y[0, 700] = [0.0, -3e16, 0.0]
    _same(X, Y, "far column")


def test_duplicates_and_open_thresholds():
    X, Y = custom(100, 2, 400, 300, sigma=0.02)
    Y = np.concatenate([Y, Y[:, :40]], axis=1)
    X = np.concatenate([X, X[:, :20]], axis=1)
    _same(X, Y, "clamp")
    _same(X, Y, "fallback", gap_mode=1)  # infinite radii
    _same(X, Y, "tau 0", tau=0.0)
