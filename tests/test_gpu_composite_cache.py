"""The composite solve's cached state is built anew where it has to be.

It is kept for the layout solved last, under other BoxArray handles too, but
its hierarchy belongs to the context's launch shapes: a knob turned between two
solves takes effect in the second, as it does for lone solves.  Seen in the
launches of the level-0 smoother: two a cycle where the level is streamed, one
per half-sweep (8) with 64-bit addresses (knob 2 off).
"""
import pytest

from test_gpu_composite import bx  # noqa: F401
from test_gpu_composite_profile import CYCLES, solve

pytestmark = pytest.mark.gpu


def test_a_turned_knob_takes_effect(bx):  # noqa: F811
    ctx = bx.default_context()
    got = []
    try:
        for knob in (1, 0, 1):
            ctx.tune(2, knob)
            got.append(solve(bx, ctx, 0))
    finally:
        ctx.tune(2, 1)
    assert [g[0] for g in got] == [2 * CYCLES, 8 * CYCLES, 2 * CYCLES]
    assert all((g[2] == got[0][2]).all() for g in got)
