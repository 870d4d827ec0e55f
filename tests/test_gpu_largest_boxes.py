"""One-box levels just below the 2 GiB that 32-bit offsets reach, periodic in
z, whose streaming kernels start several planes below the box.

A lane that must not store has the offset 2^31, and the hardware drops the
access if that is at least the box's size less the scalar offset of the
plane.  With the offset of a plane q < 0 left in place the test would be
2^31 >= bytes + |q| planes, which these boxes (2,134,440,960 bytes of 2^31 =
2,147,483,648, planes of 2.4 MB, up to 9 below) do not meet: the stores of the
planes ahead would land in the last planes.  The cell-centred results are
those of one launch per half-sweep with 64-bit addresses, to the bit (CG to
the rounding of its dots); the nodal norms, which the kernel takes in passing,
are those of the solution that it returns.
"""
import pytest

pytestmark = pytest.mark.gpu

N, PER = (768, 768, 448), (0, 0, 1)


@pytest.fixture(scope="module")
def bx():
    import paper_2403_12179_amd as bx
    return bx


def field(shape, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) * 2.0 - 1.0


def boxes(bx):
    bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in PER)
    ba = bx.BoxArray.chop((0, 0, 0), tuple(e - 1 for e in N), max(N), bc=bc)
    assert len(ba) == 1
    return ba


def past_the_end(row, planes, lead):
    """Whether dropped stores up to `lead` planes ahead would have passed."""
    plane = 8 * row
    size = 2 * plane * planes
    return size < 2 ** 31 - 128 * 8 and size + lead * plane > 2 ** 31


@pytest.mark.parametrize("par", [dict(), dict(precision=1), dict(krylov=1)])
def test_cell_centred(bx, par):
    import torch
    assert past_the_end((N[0] + 3) // 2 * (N[1] + 2), N[2] + 2, 9)
    out = []
    for knob in (1, 0):
        ctx = bx.Context(0)
        ctx.tune(2, knob)
        ba = boxes(bx)
        phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_tensor(field(N, 62))
        rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_tensor(field(N, 61))
        print("one box near 2 GiB", par, "knob", knob, flush=True)
        res = bx.mlmg_solve(phi, rhs, fixed_cycles=2, **par)
        out.append((phi.slab.clone(), res))
        del phi, rhs
    (a, ra), (b, rb) = out
    if par.get("krylov"):
        assert (a - b).abs().max() <= 1e-12 * b.abs().max()
    else:
        assert ra.hist == rb.hist and torch.equal(a, b)
    del out, a, b
    torch.cuda.empty_cache()


def test_nodal(bx):
    import torch
    assert past_the_end((N[0] + 2) // 2 * (N[1] + 1), N[2] + 1, 11)
    shape = tuple(e + 1 for e in N[::-1])  # [k, j, i]
    f, u = field(shape, 63), torch.zeros(shape, device="cuda", dtype=torch.float64)
    f[N[2]] = f[0]
    print("nodal level near 2 GiB", flush=True)
    res = bx.nodal_solve(boxes(bx), u, f, fixed_cycles=2)
    inner = (slice(0, N[2]), slice(1, -1), slice(1, -1))
    c = u[:-1]  # one period of planes
    r = torch.roll(c, 1, 0) + torch.roll(c, -1, 0) - 6.0 * c
    r[:, 1:-1] += c[:, :-2] + c[:, 2:]
    r[:, :, 1:-1] += c[:, :, :-2] + c[:, :, 2:]
    r = (f[inner] - r[:, 1:-1, 1:-1] * float(N[0]) ** 2).abs().max() / f[inner].abs().max()
    assert res.hist[-1] == pytest.approx(float(r), rel=1e-6)
    torch.cuda.empty_cache()
