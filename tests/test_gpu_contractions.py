"""The modal contractions' open schedules (the kernels that stage nothing for
few rows, and the phase blocks of fewer pixel tiles) give the sums of the
staged blocks bit for bit, at the edges of their tiles and of their rules."""

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

TWO = ((0, 0.0), (0, 1.0))
# N, P, J, M, channels, lambda_0 / lambda
CASES = [(64, 1, 1, 1, ((0, 0.0),), None), (64, 1, 17, 16, TWO, None), (64, 3, 5, 33, TWO, (1.0, 0.9)),
         (64, 2, 2, 256, ((0, 0.0),), None), (64, 8, 16, 47, TWO, None), (64, 43, 3, 20, TWO, None),
         (64, 86, 3, 48, TWO, None), (64, 75, 10, 256, ((0, 0.0),), None),
         (64, 76, 10, 256, ((0, 0.0),), None), (96, 1, 3, 17, TWO, None), (96, 26, 5, 66, TWO, (1.0, 0.9)),
         (128, 1, 2, 150, TWO, (1.0, 0.95)), (128, 13, 10, 9, TWO, None)]


@pytest.mark.parametrize("N,P,J,M,channels,lam", CASES)
def test_open_schedules_equal_staged(N, P, J, M, channels, lam):
    from paper_2505_10639_amd import Plan
    dev = torch.device("cuda:0")
    pr = synth.make_problem(140, N=N, P=1, J=1, M=M, channels=channels, lam_ratios=lam, border=6)
    plan = Plan(N, P, J, pr.channel_object, pr.pupil, pr.basis, pr.diversity, dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(N + M)
    alpha = 0.3 * torch.randn((P, J, M), generator=gen, device=dev)
    D = torch.fft.rfft2(1.0 + 0.1 * torch.randn((P, plan.C, J, N, N), generator=gen, device=dev))
    D = D.contiguous()
    open_ = plan.tuning()
    print(f"[open] N={N} P={P} J={J} M={M} {open_}", flush=True)
    l0, g0 = (t.clone() for t in plan.loss_grad(alpha, D, 1e-3))
    assert bool(torch.isfinite(g0).all()) and float(g0.abs().max()) > 0
    for row_tiles, phase in ((4, (4, 8)), (3, (4, 8)), (2, (4, 8))):
        plan.set_tuning(0, 1, 1, 4, open_["grad_splits"], row_tiles, *phase)
        l1, g1 = plan.loss_grad(alpha, D, 1e-3)
        assert torch.equal(l1, l0) and torch.equal(g1, g0), (row_tiles, phase)
    plan.close()
