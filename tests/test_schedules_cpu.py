"""Launch schedules as momfbd_tuning states them, without a device: what
get_tuning reports restores what ran, on the plan itself and on another, and
every selectable shape is the one that launches."""

import ctypes
import itertools

import pytest

from test_hostemu_cpu import emu  # noqa: F401

FIELDS = ("xcd_forward", "xcd_adjoint", "object_pairs_per_thread", "grad_waves", "grad_splits",
          "grad_row_tiles", "phase_col_tiles", "phase_waves", "object_fused")
# N, P, C, J, M, bases: columns P J on both sides of 128 and 256, rows x mode
# tiles on both sides of 12 000, modes on both sides of 160
PLANS = [(64, 1, 2, 8, 44, 1), (64, 8, 1, 16, 160, 1), (64, 43, 2, 3, 161, 1),
         (128, 16, 3, 16, 256, 3), (64, 2, 2, 128, 9, 1), (96, 257, 2, 1, 150, 1),
         (64, 750, 2, 1, 256, 1), (64, 751, 2, 1, 256, 1), (64, 961, 2, 12, 66, 1),
         (128, 128, 4, 24, 150, 4)]


def schedule(emu, plan, values=None):  # noqa: F811
    got, runs = (ctypes.c_int * 9)(), (ctypes.c_int * 7)()
    v = None if values is None else (ctypes.c_int * 9)(*values)
    ok = emu.emu_schedule((ctypes.c_int * 6)(*plan), v, got, runs)
    return (dict(zip(FIELDS, got)), tuple(runs)) if ok else None


def selectable(plan):
    grads = [(4, 0), (4, 2), (4, 3), (4, 4), (8, 0), (8, 2)]
    phases = [(0, 0), (4, 8)] + ([(8, 8), (8, 16)] if plan[4] <= 160 else [(2, 4)])
    return itertools.product((0, 1), (0, 1), (1, 2, 4), grads, (0, 1, 2, 4, 8), phases, (0, 1))


@pytest.mark.parametrize("plan", PLANS)
def test_reported_schedule_restores_what_ran(emu, plan):  # noqa: F811
    default = schedule(emu, plan)
    for xf, xa, ppt, (waves, rt), splits, (ct, pw), fused in selectable(plan):
        first = schedule(emu, plan, (xf, xa, ppt, waves, splits, rt, ct, pw, fused))
        assert first is not None, (plan, waves, rt, ct, pw)
        again = schedule(emu, plan, [first[0][f] for f in FIELDS])
        assert again == first, (plan, waves, rt, ct, pw)
        # an open shape is the plan's own choice, a selected one what was asked for
        if waves == 4 and rt in (0, 4):
            assert first[1][:3] == default[1][:3]
        else:
            assert first[1][:3] == (1, waves, rt or 2)
        if (ct, pw) in ((4, 8), (8, 16)):
            assert first[1][4:] == (1, ct, pw)
        else:
            assert first[1][4:] == default[1][4:]


def test_open_schedule_stays_open_on_another_plan(emu):  # noqa: F811
    for a, b in itertools.product(PLANS, PLANS):
        if (a[4] > 160) != (b[4] > 160):
            continue               # the pair that stands for the open phase differs
        reported, _ = schedule(emu, a)
        want, ran = schedule(emu, b)
        got, runs = schedule(emu, b, [dict(reported, grad_splits=0)[f] for f in FIELDS])
        assert (got, runs) == (want, ran), (a, b)


@pytest.mark.parametrize("plan", PLANS)
def test_refused_schedules(emu, plan):  # noqa: F811
    ok = [0, 1, 1, 4, 0, 0, 0, 0, 0]
    assert schedule(emu, plan, ok) is not None
    wide = plan[4] <= 160
    bad = [(0, 2), (2, 3), (3, 5), (4, 3), (5, 1), (5, 5), (6, 8), (8, 2)]
    for i, v in bad:
        values = list(ok)
        values[i] = v
        assert schedule(emu, plan, values) is None, (i, v)
    for ct, pw in ((4, 4), (8, 0), (0, 8), (16, 8)) + (((2, 4),) if wide else ((8, 8), (8, 16))):
        assert schedule(emu, plan, ok[:6] + [ct, pw, 0]) is None, (ct, pw)
    for rt in (3, 4):
        assert schedule(emu, plan, [0, 1, 1, 8, 0, rt, 0, 0, 0]) is None
