"""Stage timings during a composite solve: the level-0 launches of the coarse
correction's V-cycles are counted, two a cycle where the level is streamed, and
timing changes no result."""
import ctypes as C

import pytest

import workloads as W
from test_gpu_composite import bx  # noqa: F401

pytestmark = pytest.mark.gpu

N, CYCLES = 64, 3


def solve(bx, ctx, stage=-1):  # noqa: F811
    """On new handles: level-0 launches of the stage, their time, the coarse solution."""
    _, fb = W.composite_layout(N, "centre", max_box=32)
    cba = bx.BoxArray.chop((0, 0, 0), (N - 1,) * 3, 32)
    fba = bx.BoxArray.from_boxes((0, 0, 0), (2 * N - 1,) * 3, fb)
    pc, pf = bx.MultiFab(cba, ctx=ctx), bx.MultiFab(fba, ctx=ctx)
    rc = bx.MultiFab(cba, nghost=0, ctx=ctx).from_global(W.uniform_rhs((N,) * 3, 81))
    rf = bx.MultiFab(fba, nghost=0, ctx=ctx).from_global(W.uniform_rhs((2 * N,) * 3, 82))
    lib, chk = bx._lib.lib(), bx._lib.check
    chk(lib.bxmg_profile_stage(ctx._h, stage))
    chk(lib.bxmg_profile_read(ctx._h, None, None, 1))
    try:
        bx.composite_solve(pc, rc, pf, rf, fixed_cycles=CYCLES)
        n, ms = C.c_int64(), C.c_double()
        chk(lib.bxmg_profile_read(ctx._h, C.byref(n), C.byref(ms), 1))
    finally:
        chk(lib.bxmg_profile_stage(ctx._h, -1))
    return n.value, ms.value, pc.to_global()


def test_timed_stage(bx):  # noqa: F811
    ctx = bx.default_context()
    n, ms, u = solve(bx, ctx, 0)
    assert n == 2 * CYCLES and 0.0 < ms < 1e3
    assert (u == solve(bx, ctx)[2]).all()
