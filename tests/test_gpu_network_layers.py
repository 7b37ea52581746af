"""The warm-start network's layers at the edges of their tiles (frames not a
multiple of four, one burst, bursts that leave tiles part empty, every patch
size) against the FP64 oracle network on the values the kernels read."""

import numpy as np
import pytest

import synth
from helpers import fast_simulate_D
from oracle import cnn

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = [(64, 1, 9, 1), (64, 3, 10, 5), (64, 5, 13, 17), (64, 8, 66, 3), (64, 64, 9, 2),
         (96, 2, 11, 3), (96, 7, 20, 2), (128, 4, 9, 3), (128, 9, 10, 1)]


def layers(N, J, M):
    return [("conv", J, 32), ("conv", 32, 64), ("conv", 64, 128), ("conv", 128, 128),
            ("dense", 128 * (N // 16) ** 2, 512), ("dense", 512, J * M)]


def setup(N, J, M, B):
    from paper_2505_10639_amd import WarmStartNet
    dev = torch.device("cuda:0")
    pr = synth.make_problem(90, N=N, P=B, J=J, M=M, d_over_r0=np.linspace(5.0, 15.0, B),
                            border=N // 10)
    D = torch.from_numpy(fast_simulate_D(pr)).to(dev)
    onet = cnn.Network(layers(N, J, M))
    rng = np.random.default_rng(91)
    params = np.concatenate([v for kind, a, b in onet.layers for k in [9 * a if kind == "conv" else a]
                             for v in (rng.standard_normal(b * k) * np.sqrt(2.0 / k),
                                       0.05 * rng.standard_normal(b))]).astype(np.float32)
    scale = np.linspace(1.0, 0.2, M).astype(np.float32)
    net = WarmStartNet(J, M, scale, batch_max=B, device=dev, N=N)
    net.load(torch.from_numpy(params).to(dev))
    return net, onet, params.astype(np.float64), scale, D


@pytest.mark.parametrize("N,J,M,B", CASES)
def test_prediction(N, J, M, B):
    net, onet, params, scale, D = setup(N, J, M, B)
    print(f"[layers] predict N={N} J={J} M={M} B={B}", flush=True)
    pred = net.predict(D).cpu().numpy()
    x = net.input(D).cpu().numpy().astype(np.float64)
    ref = onet.forward(x, params, bf16=True)[0][-1].reshape(B, J, M) * scale
    # five layers round their activations to bfloat16; where FP32 and FP64
    # sums round to neighbouring values each adds at most 2^-8
    assert np.linalg.norm(pred - ref) <= 5 * 2.0 ** -8 * np.linalg.norm(ref)
    net.close()


@pytest.mark.parametrize("N,J,M,B", CASES)
def test_gradients(N, J, M, B):
    net, onet, params, scale, D = setup(N, J, M, B)
    print(f"[layers] gradients N={N} J={J} M={M} B={B}", flush=True)
    x = net.input(D).cpu().numpy().astype(np.float64)
    even = cnn.even_mode_mask(M)
    p = onet.forward(x, params, bf16=True)[0][-1].reshape(B, J, M)
    # twice the prediction, flipped on every third frame: the choice between a
    # frame's target and its flip is clear, and no residual is a small
    # difference of large numbers
    flip = np.where((np.arange(J) % 3 == 0)[None, :, None] & even[None, None, :], -1.0, 1.0)
    target = (2.0 * p * flip * scale).astype(np.float32)
    wt = scale.astype(np.float64) ** 2 / np.mean(scale.astype(np.float64) ** 2)
    loss, grad = net.loss_grad(D, torch.from_numpy(target).to(D.device))
    loss, grad = float(loss.cpu()[0]), grad.cpu().numpy()
    l_o, g_o, _ = onet.loss_grad(x, params, target / scale, even, bf16=True, weight=wt)
    # 2^-8 for every bfloat16 rounding point of the forward and backward pass
    # that a layer's gradient has behind it: 12 for the first three layers, 8
    # for the last three
    assert abs(loss - l_o) <= 2 * 5 * 2.0 ** -8 * l_o
    errs, o = [], 0
    for li, (kind, a, b) in enumerate(onet.layers):
        n = b * (9 * a if kind == "conv" else a) + b
        errs.append(np.linalg.norm(grad[o:o + n] - g_o[o:o + n]) / np.linalg.norm(g_o[o:o + n]))
        o += n
    print("[layers] errors", [f"{e:.1e}" for e in errs], flush=True)
    assert all(e <= (12 if li < 3 else 8) * 2.0 ** -8 for li, e in enumerate(errs)), errs
    net.close()
