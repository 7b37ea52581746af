"""Outputs that share memory with inputs which the call has read before it
writes them."""

import numpy as np
import pytest

import synth
from helpers import simulate_D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,P,J,channels", [
    (64, 3, 1, ((0, 0.0),)), (64, 2, 2, ((0, 0.0), (1, 0.0))), (96, 2, 2, ((0, 0.0),)),
    (128, 2, 1, ((0, 0.0), (1, 0.0))), (64, 2, 3, ((0, 0.0),))])
def test_filtered_objects_over_their_data(N, P, J, channels):
    """obj over D: written by the last launch only, also where the frames are
    too few (under three per object) for the workspace to hold the ratios."""
    from paper_2505_10639_amd import Plan, _lib, filter_spec
    dev = torch.device("cuda:0")
    pr = synth.make_problem(300 + N + J, N=N, P=P, J=J, M=9, channels=channels,
                            d_over_r0=np.linspace(6.0, 9.0, P))
    D = torch.from_numpy(simulate_D(pr)).to(dev)
    alpha = torch.from_numpy(pr.alpha_true).to(dev)
    plan = Plan(N, P, J, pr.channel_object, pr.pupil, pr.basis, pr.diversity, dev)
    eta = 1e-4 * float(np.sum(pr.window.astype(np.float64) ** 2))
    spec = [filter_spec("scharmer", noise_power=eta)] * pr.K
    ref, H = plan.object_filtered(alpha, D, spec, want_H=True)
    assert float(H.max()) > 0 and bool(torch.isfinite(ref).all())
    over = D.clone()
    obj = torch.view_as_real(over).reshape(-1)[:ref.numel()].view(ref.shape)
    H1 = torch.empty_like(H)
    _lib.momfbd_object_filtered(plan.handle, alpha, over, None, 1e-3, None, spec, obj, H1, plan.ws)
    assert torch.equal(H1, H) and torch.equal(obj, ref)
    plan.close()
