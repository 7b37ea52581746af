"""A tuning that get_tuning reports restores what ran, on the plan and on
another; the selectable phase blocks give the open schedule's results bit for
bit on both sides of the columns and modes where the open one changes."""

import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def make(P, J, M):
    from paper_2505_10639_amd import Plan
    dev = torch.device("cuda:0")
    pr = synth.make_problem(141, N=64, P=1, J=1, M=M, channels=((0, 0.0), (0, 1.0)), border=6)
    return Plan(64, P, J, pr.channel_object, pr.pupil, pr.basis, pr.diversity, dev)


def test_reported_tuning_round_trip():
    plans = [make(1, 9, 30), make(30, 10, 60), make(1, 2, 200), make(50, 6, 161)]
    defaults = [p.tuning() for p in plans]
    for p, t in zip(plans, defaults):
        p.set_tuning(**t)
        assert p.tuning() == t
    # the open schedule of one plan leaves another's open
    for a, b in ((0, 1), (1, 0), (2, 3), (3, 2)):
        plans[b].set_tuning(**dict(defaults[a], grad_splits=0))
        assert plans[b].tuning() == defaults[b], (defaults[a], defaults[b])
    # the phase pair that has stood for the open schedule from 161 modes on
    for p in plans[2:]:
        p.set_tuning(0, 1, 1, 4, 0, 0, 2, 4)
    for p in plans[:2]:
        with pytest.raises(Exception):
            p.set_tuning(0, 1, 1, 4, 0, 0, 2, 4)
    for p in plans:
        p.close()


@pytest.mark.parametrize("P,J,M", [(1, 1, 1), (8, 16, 47), (43, 3, 20), (8, 16, 160), (43, 3, 160),
                                   (8, 16, 161), (43, 3, 256), (90, 10, 208), (90, 10, 224),
                                   (90, 10, 240), (200, 16, 200), (200, 16, 256)])
def test_selected_shapes_equal_open(P, J, M):
    plan = make(P, J, M)
    dev = plan.device
    gen = torch.Generator(device=dev)
    gen.manual_seed(P + M)
    alpha = 0.3 * torch.randn((P, J, M), generator=gen, device=dev)
    D = torch.fft.rfft2(1.0 + 0.1 * torch.randn((P, plan.C, J, 64, 64), generator=gen, device=dev))
    D = D.contiguous()
    open_ = plan.tuning()
    l0, g0 = (t.clone() for t in plan.loss_grad(alpha, D, 1e-3))
    assert bool(torch.isfinite(g0).all()) and float(g0.abs().max()) > 0
    for phase in ((4, 8), (8, 16)) if M <= 160 else ((4, 8),):
        for waves, row_tiles in ((4, 2), (4, 3), (8, 2)):
            print(f"[schedules] P={P} J={J} M={M} {phase} {waves} x {row_tiles}", flush=True)
            plan.set_tuning(0, 1, 1, waves, open_["grad_splits"], row_tiles, *phase)
            t = plan.tuning()
            assert (t["phase_col_tiles"], t["phase_waves"], t["grad_row_tiles"]) == (*phase, row_tiles)
            l1, g1 = plan.loss_grad(alpha, D, 1e-3)
            assert torch.equal(l1, l0) and torch.equal(g1, g0), (phase, waves, row_tiles)
    plan.close()
