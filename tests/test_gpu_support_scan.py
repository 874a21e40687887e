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


# The origin of the products is the median of three columns, so that a stray
# point among them doesn't move it; where two of them are, or clusters lie far
# apart, the error taken off the thresholds passes them and the workgroups test
# every column exactly. The same pairs on either way.
@pytest.mark.parametrize("at", [30.0, 100.0, 300.0, 1000.0])
@pytest.mark.parametrize("cloud", ["X", "Y", "both", "two of three"])
def test_stray_points(at, cloud):
    X, Y = custom(101, 2, 700, 900, sigma=0.05)
    if cloud in ("X", "both"):
        X[:, 0] = [at, 0.0, 0.0]
    if cloud in ("Y", "both"):
        Y[:, 0] = [at, 0.1, 0.0]
    if cloud == "two of three":  # of the columns the origin is taken from
        for k in (0, 450):
            Y[:, k] = [at, 0.01 * k, 0.0]
    _same(X, Y, f"stray {cloud} at {at}")


@pytest.mark.parametrize("k", [2, 8])
@pytest.mark.parametrize("N,M", [(600, 1000), (257, 131)])
def test_clusters_far_apart(k, N, M):
    rng = np.random.default_rng(102 + k)
    X, Y = custom(102, 2, N, M, sigma=0.05)
    centres = rng.uniform(-1000.0, 1000.0, (k, 3)).astype(np.float32)
    _same(X + centres[rng.integers(0, k, N)], Y + centres[rng.integers(0, k, M)], f"{k} clusters")


# One row whose other columns all lie within a few roundings of its threshold:
# its nearest two at 1 and 1.05 set the radius, each other column has two rows
# of its own close by, so that only the row's threshold counts.
@pytest.mark.parametrize("offset", [0.0, 3.0, 40.0])
def test_pairs_at_the_threshold(offset):
    m, rng = 1500, np.random.default_rng(103)
    kappa = np.log(1e8) / np.log((m - 1) * 0.8 / 0.2)
    edge = (1.0 + 0.05 * kappa) * np.sqrt(1.0 + 1e-5 * (1.0 + kappa))
    v = rng.standard_normal((m, 3))
    v /= np.linalg.norm(v, axis=1, keepdims=True)
    centre = np.array([offset, -0.3 * offset, 0.0])

    def stored(shift, spread):
        r = edge * (1.0 + shift + spread * rng.uniform(-1.0, 1.0, m))
        r[:2] = 1.0, 1.05
        Y = v * r[:, None]
        X = np.concatenate([np.zeros((1, 3))] + [Y[2:] * s for s in (1.0 + 1e-3, 1.0 + 2.5e-3)])
        X, Y = (np.ascontiguousarray((c + centre).astype(np.float32)[None]) for c in (X, Y))
        note(f"pairs at the threshold: offset {offset} shift {shift} spread {spread}")
        return [_pairs(X, Y, scan)[1] for scan in (1, 2)]

    inside, outside = stored(-1e-3, 0.0), stored(1e-3, 0.0)
    at = stored(0.0, 3e-6 + 1e-6 * offset)  # float32 coordinates move a point by up to 6e-8 of its offset too
    for full, skip in (inside, outside, at):
        assert full == skip
    assert outside[0] < at[0] < inside[0]
