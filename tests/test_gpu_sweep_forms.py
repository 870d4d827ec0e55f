"""The streaming smoother's forms beyond the default solve, against one launch
per half-sweep (64-bit addressing, knob 2 off): first-order prolongation inside
the post-sweeps, the sums of squares that the norm sweeps take per block, and
conjugate gradients -- and that the levels are streamed at all: two launches
of the level-0 smoother a cycle instead of eight.

Iterates and max-norms are the same bits.  The sums of squares are added in
another order: chains of at most a few hundred terms and trees, so 1e-13 of
the norm (300 roundings of 1.1e-16, halved by the root).  The dots of CG are
summed as in twice the precision, to 1e-20 of their terms at these sizes, and
then rounded once: the same value however they are split, and so the same bits.
"""
import ctypes as C

import pytest

import workloads as W

pytestmark = pytest.mark.gpu

SIZES = [
    ((32, 32, 32), (1, 1, 1)),
    ((96, 48, 80), (1, 0, 1)),
    ((16, 256, 16), (0, 1, 0)),     # one block across x and z
    ((256, 16, 48), (0, 0, 1)),
    ((112, 144, 96), (0, 0, 0)),    # blocks that do not divide the domain
]


@pytest.fixture(scope="module")
def bx():
    import paper_2403_12179_amd as bx
    return bx


def boxes(bx, n, per):
    bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in per)
    return bx.BoxArray.chop((0, 0, 0), tuple(e - 1 for e in n), max(n), bc=bc)


def both(bx, n, per, beta, **par):
    """(solution, result, level-0 smoother launches) streamed and not."""
    lib, chk = bx._lib.lib(), bx._lib.check
    out = []
    for knob in (1, 0):
        ctx = bx.Context(0)
        ctx.tune(2, knob)
        ba = boxes(bx, n, per)
        phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 62))
        rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 61, mean_zero=all(per)))
        b = bx.MultiFab(ba, ctx=ctx).set_val(1.0).from_global(beta) if beta is not None else None
        chk(lib.bxmg_profile_stage(ctx._h, 0))
        res = bx.mlmg_solve(phi, rhs, b, max_cycles=6, **par)
        k, ms = C.c_int64(), C.c_double()
        chk(lib.bxmg_profile_read(ctx._h, C.byref(k), C.byref(ms), 1))
        out.append((phi.to_global(), res, k.value))
    return out


def same(a, b, cycles=None):
    (ua, ra, ka), (ub, rb, kb) = a, b
    assert ra.cycles == rb.cycles and ra.status == rb.status
    assert kb == 4 * ka and (cycles is None or ka == 2 * ra.cycles)
    assert ra.hist == rb.hist and (ua == ub).all()
    assert ra.hist_l2 == pytest.approx(rb.hist_l2, rel=1e-13, abs=0.0)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,per", SIZES)
def test_first_order_prolongation(bx, n, per, precision):
    a, b = both(bx, n, per, None, precision=precision, prolong=1)
    same(a, b, cycles=True)
    second, _ = both(bx, n, per, None, precision=precision)
    assert second[1].hist != a[1].hist  # (another interpolation)


@pytest.mark.parametrize("n,per", SIZES)
def test_first_order_prolongation_varcoef(bx, n, per):
    beta = 10.0 ** W.uniform_rhs(n, 63) ** 3 * 10.0 ** (2 * W.uniform_rhs(n, 64))
    same(*both(bx, n, per, beta, precision=1, prolong=1), cycles=True)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,per", SIZES)
def test_sums_of_squares(bx, n, per, precision):
    same(*both(bx, n, per, None, precision=precision), cycles=True)
    same(*both(bx, n, per, None, precision=precision, alpha=977.25), cycles=True)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,per", SIZES)
def test_cg_bits(bx, n, per, precision):
    same(*both(bx, n, per, None, precision=precision, krylov=1))


@pytest.mark.parametrize("n,per", SIZES)
def test_cg_bits_varcoef(bx, n, per):
    beta = W.smooth_gaussian_beta(n, 65)
    same(*both(bx, n, per, beta, precision=1, krylov=1))


@pytest.mark.parametrize("per", [(1, 1, 1), (1, 0, 1)])
def test_first_order_prolongation_batch(bx, per):
    sizes = [(32, 32, 32), (96, 48, 80), (64, 64, 64), (16, 128, 32)]
    out = []
    for knob in (1, 0):
        ctx = bx.Context(0)
        ctx.tune(2, knob)
        b = bx.Batch(ctx, 64 << 20, 4, precision=1, max_cycles=7, prolong=1)
        probs = {}
        for q, n in enumerate(sizes):
            ba = boxes(bx, n, per)
            phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0)
            rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 70 + q, mean_zero=all(per)))
            probs[b.add(phi, rhs)] = (q, phi, rhs)
        assert None not in probs
        res = {probs[i][0]: (probs[i][1].to_global(), r) for i, r in b.run(2)}
        b.close()
        out.append(res)
    for q in range(len(sizes)):
        (ua, ra), (ub, rb) = out[0][q], out[1][q]
        assert (ra.cycles, ra.status, ra.hist) == (rb.cycles, rb.status, rb.hist)
        assert ra.hist_l2 == pytest.approx(rb.hist_l2, rel=1e-13, abs=0.0)
        assert (ua == ub).all(), q
