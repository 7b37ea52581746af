"""The object pass that leaves the Loefdahl-Scharmer ratios: whole groups of six
frames and remainders, weights, a gamma table, and the ratios in either of their
two places (fewer than three frames per object).  The filter is compared with
the oracle's from the OTFs that the device computed: the ratio does not depend
on the scale of the OTFs, so near and beyond the diffraction limit their
roundings decide it."""

import numpy as np
import pytest

import oracle
import synth
from helpers import OBJ_RMS, simulate_D
from oracle import postprocess as pp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,P,J,M,channels", [
    (64, 1, 1, 6, ((0, 0.0),)), (96, 1, 2, 12, ((0, 0.0), (1, 0.0))),
    (64, 2, 6, 10, ((0, 0.0), (0, 1.0))), (64, 2, 7, 10, ((0, 0.0), (1, 0.0))),
    (128, 1, 13, 8, ((0, 0.0),))])
def test_scharmer_ratios(N, P, J, M, channels):
    from paper_2505_10639_amd import Plan, filter_spec
    dev = torch.device("cuda:0")
    pr = synth.make_problem(N + J, N=N, P=P, J=J, M=M, channels=channels,
                            d_over_r0=np.linspace(6.0, 10.0, P))
    D_np = simulate_D(pr)
    w = np.random.default_rng(J).uniform(0.5, 2.0, (pr.C, J)).astype(np.float32)
    g0, lam = [1e-3] * pr.K, [0.05] * pr.K
    # FP32, as the library takes it
    eta = float(np.float32(1.1e-4 * float(np.sum(pr.window.astype(np.float64) ** 2))))
    plan = Plan(N, P, J, pr.channel_object, pr.pupil, pr.basis, pr.diversity, dev)
    alpha, D = torch.from_numpy(pr.alpha_true).to(dev), torch.from_numpy(D_np).to(dev)
    obj, H = plan.object_filtered(alpha, D, [filter_spec("scharmer", noise_power=eta)] * pr.K,
                                  plan.smoothness_gamma(g0, lam), torch.from_numpy(w).to(dev),
                                  want_H=True)
    S = plan.forward(alpha, want_psf=False, want_otf=True)[1]
    torch.cuda.synchronize()
    obj, H, S = obj.cpu().numpy(), H.cpu().numpy(), S.cpu().numpy()
    for p in range(P):
        r = oracle.evaluate_patch(pr.alpha_true[p], D_np[p], pr.basis, pr.diversity, pr.pupil,
                                  pr.channel_object, oracle.smoothness_gamma(N, g0, lam), weights=w,
                                  want_grad=False)
        Df = oracle.expand_half(D_np[p], N)
        Sf = oracle.expand_half(S[p], N)
        for k in range(pr.K):
            chans = [c for c in range(pr.C) if pr.channel_object[c] == k]
            # FP64 sums of the same FP32 numbers: the clip decision is the same
            # on both sides unless a ratio lies at the threshold
            assert np.min(np.abs(pp.scharmer_raw(Df, Sf, w, chans, eta) - 0.2)) > 1e-9
            Hk = pp.scharmer_filter(Df, Sf, w, chans, eta)
            half = Hk[:, :N // 2 + 1]
            assert 0 < np.count_nonzero(Hk) < Hk.size // 2
            np.testing.assert_array_equal(H[p, k] > 0, half > 0)
            np.testing.assert_allclose(H[p, k], half, rtol=2.0 ** -23, atol=0)
            ref = pp.filtered_object(r["O"][k], Hk)
            assert np.sqrt(np.mean((obj[p, k] - ref) ** 2)) < OBJ_RMS, (p, k)
    plan.close()
