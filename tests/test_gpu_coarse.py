"""The fused coarse cycle in registers and LDS against the one on device memory.

Knob 4 off keeps the coarse levels in device memory.  Both forms take every
cell's arithmetic and every sum of the bottom's conjugate gradients in the
same order, so solves give the same bits.  The sizes reach each form of the
bottom: one wave of one or two cells per lane, one cell per thread, and a
bottom alone of several cells per thread; levels of one wave and of the
workgroup; odd bottoms, mixed boundaries, both precisions and coefficients.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bx():
    import paper_2403_12179_amd as bx
    return bx


def solve(bx, n, per, var, knob, **par):
    ctx = bx.Context(0)
    ctx.tune(4, knob)
    bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in per)
    ba = bx.BoxArray.chop((0, 0, 0), tuple(e - 1 for e in n), max(n), bc=bc)
    phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0)
    rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 71, mean_zero=all(per)))
    beta = bx.MultiFab(ba, ctx=ctx).set_val(1.0).from_global(W.smooth_gaussian_beta(n, 72)) if var else None
    res = bx.mlmg_solve(phi, rhs, beta, fixed_cycles=3, **par)
    return phi.to_global(), res


@pytest.mark.parametrize("n,per", [
    ((32, 32, 32), (1, 1, 1)),     # 16^3 ... 2^3
    ((24, 40, 20), (0, 1, 0)),     # bottom 6 x 10 x 5 = 300: one cell per thread
    ((48, 24, 40), (1, 0, 0)),     # bottom 6 x 3 x 5 = 90: two cells per lane
    ((30, 30, 30), (0, 0, 0)),     # the bottom alone, 15^3
    ((30, 22, 18), (1, 1, 1)),     # odd bottom 15 x 11 x 9, singular
    ((80, 16, 16), (0, 0, 1)),     # 40 x 8 x 8 ... 5 x 1 x 1
    ((16, 128, 16), (0, 0, 0)),    # a top level 2 pairs wide after two coarsenings
])
@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("precision", [0, 1])
def test_lds_equals_device_memory(bx, n, per, var, precision):
    for par in (dict(), dict(nu1=0, nu2=1, prolong=1), dict(nu1=1, nu2=3, alpha=55.5)):
        a, ra = solve(bx, n, per, var, 1, precision=precision, **par)
        b, rb = solve(bx, n, per, var, 0, precision=precision, **par)
        assert ra.hist == rb.hist
        assert (a == b).all()
