"""A patch's spectrum does not depend on how many patches are cut with it (64 x
64: one unit to a workgroup up to 4096 units, four beyond)."""

import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,n,J", [(64, 1, 4095), (64, 8, 64), (64, 13, 25), (96, 3, 5), (128, 2, 3)])
def test_spectra_of_many_and_few_patches_agree(N, n, J):
    from paper_2505_10639_amd import Plan
    dev = torch.device("cuda:0")
    pr = synth.make_problem(151, N=N, P=1, J=1, M=1, border=N // 10)
    win = torch.from_numpy(pr.window).to(dev)
    gen = torch.Generator(device=dev)
    gen.manual_seed(N + n)
    # one frame more than the patches of J frames fill
    side = N + 7 * (n - 1)
    frames = 1.0 + 0.1 * torch.randn((1, J + 2, side, side), generator=gen, device=dev)
    many = Plan(N, n * n, J + 2, [0], pr.pupil[:1], pr.basis[:1], None, dev)
    one = Plan(N, n * n, 1, [0], pr.pupil[:1], pr.basis[:1], None, dev)
    D = many.prepare_data(frames, 7, win)
    for j in (0, J // 2, J + 1):
        Dj = one.prepare_data(frames[:, j:j + 1].contiguous(), 7, win)
        assert torch.equal(Dj[:, :, 0], D[:, :, j]), j
    many.close()
    one.close()
