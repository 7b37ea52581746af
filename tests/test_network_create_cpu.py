"""Network creation without a device: the sizes are formed for every batch the
call accepts."""

import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CREATE = """
import ctypes, sys, numpy as np
from paper_2505_10639_amd import _lib
scale, out = np.ones(8, np.float32), ctypes.c_void_p()
st = _lib.lib().momfbd_cnn_create(int(sys.argv[1]), 1, 8, int(sys.argv[2]),
                                  scale.ctypes.data_as(ctypes.c_void_p), ctypes.byref(out))
print("status", st)
"""


@pytest.mark.parametrize("N", [64, 96, 128])
@pytest.mark.parametrize("batch_max", [1, 256, 1 << 19, 1 << 22, 2 ** 31 - 1])
def test_create_for_any_batch(N, batch_max):
    # in a child process: an arithmetic fault there is an exit status here
    r = subprocess.run([sys.executable, "-c", CREATE, str(N), str(batch_max)], capture_output=True,
                       text=True, cwd=ROOT, timeout=60)
    # 0 with a device; without one the first device call fails
    assert r.returncode == 0 and r.stdout.strip() in ("status 0", "status -4"), r
