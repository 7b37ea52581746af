"""The order of the patch cuts, without a device: every unit is cut exactly
once, and each of the 8 XCDs takes a contiguous run of the frames' order."""

import ctypes

import pytest

from test_hostemu_cpu import emu  # noqa: F401


@pytest.mark.parametrize("per_block", [1, 4])
def test_every_unit_once(emu, per_block):  # noqa: F811
    for units in list(range(1, 140)) + [255, 256, 257, 4095, 4096, 4097, 4100, 23064]:
        cap = units + 64 * per_block
        out = (ctypes.c_int * cap)()
        blocks = emu.emu_cut_order(units, per_block, out, cap)
        assert blocks % 8 == 0 and (blocks - 8) * per_block < units
        cut = [out[b] * per_block + w for b in range(blocks) for w in range(per_block)]
        assert sorted(u for u in cut if u < units) == list(range(units)), units
        for xcd in range(8):
            run = [out[b] for b in range(xcd, blocks, 8)]
            assert run == list(range(run[0], run[0] + len(run)))
