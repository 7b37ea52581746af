"""Weight and bias gradients of every layer, each on its own, over the frame
counts at which the first layer's kernels change (14/15, 16, 28/29), against
the FP64 oracle network on the values the kernels read."""

import numpy as np
import pytest

from oracle import cnn
from test_gpu_network_layers import setup as make_net

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,J,M,B", [(64, 14, 9, 3), (64, 15, 12, 4), (64, 16, 9, 2), (64, 28, 9, 3),
                                     (64, 29, 10, 2), (96, 24, 9, 2), (128, 27, 8, 1)])
def test_gradients_by_tensor(N, J, M, B):
    net, onet, params, scale, D = make_net(N, J, M, B)
    print(f"[frames] gradients N={N} J={J} M={M} B={B}", flush=True)
    x = net.input(D).cpu().numpy().astype(np.float64)
    even = cnn.even_mode_mask(M)
    p = onet.forward(x, params, bf16=True)[0][-1].reshape(B, J, M)
    # twice the prediction, flipped on every third frame: a clear choice
    # between a frame's target and its flip
    flip = np.where((np.arange(J) % 3 == 0)[None, :, None] & even[None, None, :], -1.0, 1.0)
    target = (2.0 * p * flip * scale).astype(np.float32)
    wt = scale.astype(np.float64) ** 2 / np.mean(scale.astype(np.float64) ** 2)
    _, grad = net.loss_grad(D, torch.from_numpy(target).to(D.device))
    grad = grad.cpu().numpy()
    _, g_o, _ = onet.loss_grad(x, params, target / scale, even, bf16=True, weight=wt)
    # 2^-8 for every bfloat16 rounding point that a layer's gradient has behind
    # it: 12 for the first three layers, 8 for the last three.  A bias gradient
    # is the plain sum of the rows that the weight gradient weighs: roundings
    # and rows add alike, so the bound is the same.
    errs, o = [], 0
    for li, (kind, a, b) in enumerate(onet.layers):
        for name, n in (("w", b * (9 * a if kind == "conv" else a)), ("b", b)):
            errs.append((li, name, np.linalg.norm(grad[o:o + n] - g_o[o:o + n]) /
                         np.linalg.norm(g_o[o:o + n])))
            o += n
    print("[frames] errors", [f"{li}{n} {e:.1e}" for li, n, e in errs], flush=True)
    assert all(e <= (12 if li < 3 else 8) * 2.0 ** -8 for li, n, e in errs), errs
    net.close()
