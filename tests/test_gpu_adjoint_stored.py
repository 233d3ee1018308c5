"""Gradients of lattices on both sides of the line between the kernels that
store the adjoint's states (packs up to three slots per thread, tiles beyond),
against the oracle's gradient; the tolerance is the one of the smaller ones'."""
import numpy as np
import pytest

from tests.test_gpu_adjoint import _oracle_w, _setup, ft  # noqa: F401 (ft: the fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind,a,b", [("torus", 5, 9), ("hex", 4, 0)])
def test_gradient_of_stored_runs(ft, orc, kind, a, b):  # noqa: F811
    import torch
    dt, steps, re, ckpt, U = 0.02, 12, 6, 5, 2.5
    olat, rho0, prob = _setup(ft, orc, kind, a, b, "neel", 4, 5, "f32")
    target, w = _oracle_w(orc, olat, rho0, dt, steps, re, U)
    _, gU, gt, gs = orc.occupation_loss_grad(olat, U, rho0, dt, steps, re, target)
    ref = np.concatenate([[gU, gt], gs.reshape(-1)])
    grad, _ = ft.adjoint(prob, dt, steps, re, ckpt, torch.from_numpy(w).cuda())
    torch.cuda.synchronize()
    assert np.max(np.abs(grad.cpu().numpy() - ref)) <= 2e-3 * np.max(np.abs(ref))
