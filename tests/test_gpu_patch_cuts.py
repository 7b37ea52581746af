"""Patch cuts in the frame-by-frame order (units that leave a workgroup or an
XCD's run part empty, odd strides and widths), and the generator's unaligned
output."""

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("N,ny,nx,stride,extra,J,channels", [
    (64, 1, 1, 64, 0, 1, ((0, 0.0),)), (64, 1, 3, 17, 5, 3, ((0, 0.0),)),
    (64, 3, 5, 33, 2, 3, ((0, 0.0), (1, 0.0))), (96, 1, 1, 96, 0, 1, ((0, 0.0),)),
    (96, 2, 3, 31, 7, 3, ((0, 0.0),)), (128, 1, 2, 65, 1, 5, ((0, 0.0),)),
    (128, 2, 2, 128, 3, 1, ((0, 0.0), (1, 0.0)))])
def test_prepare_data(N, ny, nx, stride, extra, J, channels):
    from paper_2505_10639_amd import Plan
    dev = torch.device("cuda:0")
    pr = synth.make_problem(150, N=N, P=1, J=1, M=3, channels=channels, border=N // 10)
    H, W = (ny - 1) * stride + N, (nx - 1) * stride + N + min(extra, stride - 1)
    rng = np.random.default_rng(N + nx)
    frames = (1.0 + 0.1 * rng.standard_normal((len(channels), J, H, W))).astype(np.float32)
    plan = Plan(N, ny * nx, J, pr.channel_object, pr.pupil, pr.basis, None, dev)
    D = plan.prepare_data(torch.from_numpy(frames).to(dev), stride, torch.from_numpy(pr.window).to(dev))
    ref = oracle.prepare_data(frames.astype(np.float64), pr.window, N, stride)
    d = D.cpu().numpy() - ref
    # FP32: the mean, window and 2 log2 N butterfly stages, 2^-24 each, on
    # spectra whose norm the mean dominates
    assert np.linalg.norm(d) <= (4 + 2 * np.log2(N)) * 2.0 ** -24 * np.linalg.norm(ref)
    plan.close()


def test_normals_unaligned():
    from paper_2505_10639_amd import _lib
    dev = torch.device("cuda:0")
    a = torch.empty(1003, device=dev)
    b = torch.empty(1004, device=dev)[1:]
    _lib.momfbd_random_normal(7, 3, 0, a)
    _lib.momfbd_random_normal(7, 3, 0, b)
    assert torch.equal(a, b)
