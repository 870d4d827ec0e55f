"""The streaming smoother against one launch per half-sweep.

Both run the same arithmetic per cell in the same order, so whole solves on
them give the same bits: the iterates, the histories of max-norms and the
cycle counts are compared exactly.  The one-launch-per-half-sweep path is
the one 64-bit addressing (knob 2 off) takes.  The sizes cover domains of
one block, blocks that do not divide the domain, blocks that span it in one
direction only, the smallest levels the smoother takes and a periodic
direction narrower than a block with its halo.  Batches, whose streamed
levels run in one launch over all problems and keep their second iterate
array in the FP64 arena, are compared in the same way, with problems admitted
into ranges that others have left.
"""
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def bx():
    import paper_2403_12179_amd as bx
    return bx


def solve(bx, n, lo, per, knob, **par):
    ctx = bx.Context(0)
    ctx.tune(2, knob)
    bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in per)
    ba = bx.BoxArray.chop(lo, tuple(a + e - 1 for a, e in zip(lo, n)), max(n), bc=bc)
    f = W.uniform_rhs(n, 61, mean_zero=all(per))
    g = W.uniform_rhs(n, 62)
    phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(g)
    rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(f)
    res = bx.mlmg_solve(phi, rhs, **par)
    out = phi.to_global()
    return out, res


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("n,lo,per", [
    ((32, 32, 32), (0, 0, 0), (1, 1, 1)),
    ((32, 32, 32), (-32, 16, 0), (0, 0, 0)),
    ((96, 48, 80), (0, 0, 0), (1, 0, 1)),
    ((16, 256, 16), (0, 0, 0), (0, 1, 0)),
    ((256, 16, 48), (0, 0, 0), (0, 0, 1)),
    ((32, 16, 208), (0, 0, 0), (1, 1, 0)),
    ((112, 144, 96), (0, 0, 0), (0, 1, 0)),
    ((144, 112, 48), (0, 0, 0), (1, 0, 0)),
])
def test_streamed_equals_half_sweeps(bx, n, lo, per, precision):
    for par in (dict(), dict(alpha=977.25), dict(krylov=1)):
        a, ra = solve(bx, n, lo, per, 1, precision=precision, max_cycles=6, **par)
        b, rb = solve(bx, n, lo, per, 0, precision=precision, max_cycles=6, **par)
        assert ra.cycles == rb.cycles and ra.status == rb.status
        if not par.get("krylov"):  # (the dots of CG are summed over other tiles' partials)
            assert ra.hist == rb.hist
            assert (a == b).all()
        else:
            assert abs(a - b).max() <= 1e-9 * abs(b).max()


@pytest.mark.parametrize("n,per", [
    ((32, 32, 32), (1, 1, 1)),
    ((96, 48, 80), (0, 0, 0)),
    ((16, 256, 16), (0, 1, 0)),
    ((256, 16, 48), (0, 0, 1)),
    ((32, 16, 208), (1, 1, 0)),
    ((112, 144, 96), (1, 0, 0)),
])
def test_streamed_varcoef_equals_half_sweeps(bx, n, per):
    """Coefficients over six decades, drawn cell by cell."""
    bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in per)
    beta = 10.0 ** W.uniform_rhs(n, 63) ** 3 * 10.0 ** (2 * W.uniform_rhs(n, 64))
    f = W.uniform_rhs(n, 61, mean_zero=all(per))
    for par in (dict(), dict(alpha=977.25), dict(krylov=1)):
        out = []
        for knob in (1, 0):
            ctx = bx.Context(0)
            ctx.tune(2, knob)
            ba = bx.BoxArray.chop((0, 0, 0), tuple(e - 1 for e in n), max(n), bc=bc)
            phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 62))
            rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(f)
            bmf = bx.MultiFab(ba, ctx=ctx).set_val(1.0).from_global(beta)
            res = bx.mlmg_solve(phi, rhs, bmf, precision=1, max_cycles=5, **par)
            out.append((phi.to_global(), res))
        (a, ra), (b, rb) = out
        assert ra.cycles == rb.cycles and ra.status == rb.status
        if not par.get("krylov"):
            assert ra.hist == rb.hist
            assert (a == b).all()
        else:
            assert abs(a - b).max() <= 1e-9 * abs(b).max()


@pytest.mark.parametrize("per", [(1, 1, 1), (0, 0, 0), (1, 0, 1)])
def test_streamed_batch_equals_half_sweeps(bx, per):
    sizes = [(32, 32, 32), (96, 48, 80), (16, 16, 16), (64, 64, 64), (16, 128, 32), (32, 32, 32), (40, 24, 56)]
    out = []
    for knob in (1, 0):
        ctx = bx.Context(0)
        ctx.tune(2, knob)
        bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in per)
        b = bx.Batch(ctx, 24 << 20, 4, precision=1, max_cycles=7)
        todo, probs, res = list(range(len(sizes))), {}, {}
        while todo or len(res) < len(sizes):
            while todo:
                n = sizes[todo[0]]
                ba = bx.BoxArray.chop((0, 0, 0), tuple(e - 1 for e in n), max(n), bc=bc)
                f = W.uniform_rhs(n, 70 + todo[0], mean_zero=all(per))
                phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(W.uniform_rhs(n, 90 + todo[0]))
                rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_global(f)
                pid = b.add(phi, rhs)
                if pid is None:
                    break
                probs[pid] = (todo.pop(0), phi, rhs)
            for pid, r in b.run(2):
                q, phi, _ = probs[pid]
                res[q] = (phi.to_global(), r.cycles, r.status, r.hist)
        b.close()
        out.append(res)
    for q in range(len(sizes)):
        (ua, *ra), (ub, *rb) = out[0][q], out[1][q]
        assert ra == rb, q
        assert (ua == ub).all(), q
