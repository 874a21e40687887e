"""The reverse sweeps of larger samples exchange one word per point and phase
through memory. Where that does not fit (the static scratch of the no-alloc
entry point with many iterations), the per-iteration launches take the sweeps:
the same recurrences, summed in another order."""
import numpy as np
import pytest
import torch

import paper_2512_19743_amd as apml
from workloads import custom

from ._parity import note, rel_norm

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    apml.load()


# 2 x (4096 + 4096) points: at 600 iterations the saved scalings take 79 MB of
# the 128 MB and the exchange would take as much again; at 10 it fits
@pytest.mark.parametrize("L", [10, 600])
def test_reverse_sweeps_without_room_for_the_exchange(L):
    X, Y = custom(95, 2, 4096, 4096, reference="primitives", prediction="perm_noise", sigma=0.02)
    note(f"no-alloc reverse sweeps, L={L}")
    x, y = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
    prm = apml.apml_params_default(n_iter=L)
    gl = torch.tensor([1.0, -0.5], device="cuda")
    loss, plan = apml.apml_forward(x, y, prm)
    gx, gy = apml.apml_backward(plan, x, y, gl, want_grad_y=True)
    l2, gx2, gy2 = apml.apml_forward_backward_noalloc(x, y, prm, grad_loss=gl, want_grad_y=True)
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(loss, l2)
    # double precision on both sides: single-precision outputs agree to their rounding
    for a, b in ((gx, gx2), (gy, gy2)):
        assert rel_norm(a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)) <= 2e-7
