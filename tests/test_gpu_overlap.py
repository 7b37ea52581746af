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


@pytest.mark.parametrize("N,P,J,over", [(64, 5, 3, "noise"), (64, 5, 3, "O"), (64, 5, 3, "sigma"),
                                        (64, 1, 1, "noise"), (96, 3, 2, "noise"), (128, 2, 2, "O")])
def test_bursts_over_their_inputs(N, P, J, over):
    """D over the noise, the objects or the noise levels: the frames are whole
    before the first spectrum is written."""
    from paper_2505_10639_amd import Plan, _lib
    dev = torch.device("cuda:0")
    pr = synth.make_problem(330 + N, N=N, P=1, J=1, M=9, channels=((0, 0.0), (1, 0.0)))
    plan = Plan(N, P, J, pr.channel_object, pr.pupil, pr.basis, pr.diversity, dev)
    rng = np.random.default_rng(N + J)
    f32 = lambda *shape: torch.from_numpy(rng.standard_normal(shape).astype(np.float32)).to(dev)
    half = N * (N // 2 + 1)
    alpha, win = 0.3 * f32(P, J, 9), torch.from_numpy(pr.window).to(dev)
    ins = {"O": torch.fft.rfft2(1.0 + 0.1 * f32(P, 2, N, N)).contiguous(),
           "noise": f32(P, 2, J, N, N), "sigma": 0.01 + 0.01 * f32(P).abs()}
    frames, D = plan.synthesize(alpha, ins["O"], ins["noise"], ins["sigma"], win)
    assert bool(torch.isfinite(frames).all()) and float(D.abs().max()) > 0
    # the shared input ends where D ends
    D1 = torch.empty(P * 2 * J * half, dtype=torch.complex64, device=dev)
    src = ins[over]
    as_float = torch.view_as_real(src).reshape(-1) if src.is_complex() else src.reshape(-1)
    flat = torch.view_as_real(D1).reshape(-1)
    flat[flat.numel() - as_float.numel():] = as_float
    shared = flat[flat.numel() - as_float.numel():]
    ins[over] = (torch.view_as_complex(shared.view(-1, 2)) if src.is_complex() else shared).view(src.shape)
    frames1 = torch.empty_like(frames)
    _lib.momfbd_synthesize(plan.handle, alpha, ins["O"], ins["noise"], ins["sigma"], win, frames1,
                           D1, plan.ws)
    assert torch.equal(frames1, frames)
    # at 64 x 64 the spectra then come from another kernel: the roundings of
    # the mean, the window and 2 log2 N butterfly stages
    err = torch.linalg.vector_norm(D1.view(D.shape) - D) / torch.linalg.vector_norm(D)
    assert float(err) <= (4 + 2 * np.log2(N)) * 2.0 ** -24
    plan.close()
