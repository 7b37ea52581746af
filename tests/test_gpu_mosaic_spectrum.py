"""Mosaic at the limits of the two-patches-per-axis kernel, and the power
spectrum at every split of the merged FFT stages."""

import numpy as np
import pytest

from oracle import postprocess as pp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,ny,nx,stride,border", [
    (64, 1, 1, 64, 8), (64, 2, 9, 32, 32), (64, 3, 9, 31, 8), (64, 2, 3, 63, 0), (96, 2, 5, 48, 9),
    (96, 1, 4, 7, 12), (128, 2, 4, 64, 20)])
def test_mosaic(N, ny, nx, stride, border):
    from paper_2505_10639_amd import Plan
    import synth
    dev = torch.device("cuda:0")
    pr = synth.make_problem(70, N=N, P=1, J=1, M=3, channels=((0, 0.0), (1, 0.0)))
    plan = Plan(N, ny * nx, 1, pr.channel_object, pr.pupil, pr.basis, pr.diversity, dev)
    obj = (np.random.default_rng(N + stride).standard_normal((ny * nx, 2, N, N)) + 1).astype(np.float32)
    out = plan.mosaic(torch.from_numpy(obj).to(dev), ny, nx, stride, border).cpu().numpy()
    for k in range(2):
        ref = pp.mosaic(obj[:, k].astype(np.float64), ny, nx, stride, border)
        # FP64 sums, rounded once
        np.testing.assert_allclose(out[k], ref, rtol=2.0 ** -23, atol=2.0 ** -40)
    plan.close()


@pytest.mark.parametrize("L", [16, 32, 64, 128, 512, 1024, 2048, 4096])
@pytest.mark.parametrize("windowed", [False, True])
def test_power_spectrum(L, windowed):
    from paper_2505_10639_amd import momfbd_power_spectrum
    rng = np.random.default_rng(L)
    img = (1.0 + 0.2 * rng.standard_normal((L, L))).astype(np.float32)
    win = rng.uniform(0.0, 1.0, (L, L)).astype(np.float32) if windowed else None
    nb = min(L, L // 2 + 5)
    P, sec, cnt = momfbd_power_spectrum(torch.from_numpy(img).cuda(),
                                        None if win is None else torch.from_numpy(win).cuda(), nb)
    P, sec, cnt = P.cpu().numpy(), sec.cpu().numpy(), cnt.cpu().numpy()
    w = np.ones((L, L)) if win is None else win.astype(np.float64)
    ref = pp.power_spectrum(img.astype(np.float64), w)
    # ||dX|| <= e ||X||: six roundings per butterfly of 2 log2 L stages, and the
    # input's; |dP| <= |dX| (2 |X| + |dX|), so the 1-norms are within 2 e + e^2
    e = (12 * np.log2(L) + 4) * 2.0 ** -24
    assert np.sum(np.abs(P - ref)) <= (2 * e + e * e) * np.sum(ref)
    # the oracle's bins, 4 |u|^2 from (2 k - 1)^2 on, in closed form (its own
    # search takes L^3 steps)
    u = np.where(np.arange(L) > L // 2, np.arange(L) - L, np.arange(L))
    u2 = u * u
    k = (1 + np.floor(np.sqrt(4.0 * (u2[:, None] + u2[None, :]))).astype(int)) // 2
    sel = (k < nb) & (u2[:, None] > 0) & (u2[None, :] > 0) & (u2[:, None] <= 3 * u2[None, :]) & (
        u2[None, :] <= 3 * u2[:, None])
    count = np.bincount(k[sel], minlength=nb)
    total = np.bincount(k[sel], weights=P[sel].astype(np.float64), minlength=nb)
    np.testing.assert_array_equal(cnt, count)
    np.testing.assert_allclose(sec, total / np.maximum(count, 1), rtol=1e-12)
