"""Stage timings of lone solves: the stages that the streaming smoother takes
in (residual and norms, residual and restriction, prolongation) are launches
of their own while one of them is timed, as many as with one launch per
half-sweep (knob 2 off), and timing changes no bit of the solution."""
import ctypes as C

import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bx():
    import paper_2403_12179_amd as bx
    return bx


def launches(bx, knob, stage, var, **par):
    n = (64, 48, 32)
    ctx = bx.Context(0)
    ctx.tune(2, knob)
    ba = bx.BoxArray.chop((0, 0, 0), tuple(e - 1 for e in n), 64)
    phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0)
    rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 85))
    beta = bx.MultiFab(ba, ctx=ctx).set_val(1.0).from_global(W.smooth_gaussian_beta(n, 86)) if var else None
    lib, chk = bx._lib.lib(), bx._lib.check
    chk(lib.bxmg_profile_stage(ctx._h, stage))
    res = bx.mlmg_solve(phi, rhs, beta, **par)
    k, ms = C.c_int64(), C.c_double()
    chk(lib.bxmg_profile_read(ctx._h, C.byref(k), C.byref(ms), 1))
    return k.value, res, phi.to_global()


@pytest.mark.parametrize("var,par", [
    (False, dict(fixed_cycles=3)),
    (False, dict(precision=1, fixed_cycles=3)),
    (True, dict(precision=1, krylov=1)),
])
@pytest.mark.parametrize("stage", [1, 2, 3])
def test_stages_inside_streamed_levels(bx, stage, var, par):
    k, res, u = launches(bx, 1, stage, var, **par)
    k0, _, _ = launches(bx, 0, stage, var, **par)
    none, plain, v = launches(bx, 1, -1, var, **par)
    assert k == k0 and none == 0
    if par.get("krylov"):  # (CG takes its norms in its update)
        assert (k > 0) == (stage != 1)
        assert res.ok and abs(u - v).max() <= 1e-9 * abs(v).max()
    else:
        assert k >= 3 and (u == v).all() and res.hist == plain.hist
