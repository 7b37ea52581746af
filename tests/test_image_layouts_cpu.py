"""The 64 x 64 inverse transform through the half-size buffer and the image's
transposes to column layout and back, lane by lane on the CPU."""

import ctypes

import numpy as np

import oracle
from test_hostemu_cpu import emu, ptr, rng  # noqa: F401


def test_inverse_half_buffer_and_image_transposes(emu):  # noqa: F811
    H = oracle.dft2(rng(21).standard_normal((64, 64)))
    half = H[:, :33].astype(np.complex64)
    out = np.zeros((64, 64), np.float32)
    emu.emu_c2r_half(ptr(half.view(np.float32)), ptr(out))
    ref = oracle.idft2_un(oracle.expand_half(half, 64)).real
    # the full-buffer form's bound; NaN marks a value that did not come back
    assert np.abs(out - ref).max() <= 5e-7 * np.abs(ref).max()
