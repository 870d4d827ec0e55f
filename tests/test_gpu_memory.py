"""Solves on a device with room for what they cannot do without, but not for the
streamed levels' second arrays: they run those levels one launch per half-sweep
and give the same results.  Each solve is run with room first, the second time
(the runtime's own allocations done) to see what it allocates; then tensors
take the rest of the device but for that less half of level 0's second array."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu

N = 384


@pytest.fixture(scope="module")
def bx():
    import paper_2403_12179_amd as bx
    return bx


def free():
    import torch
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()[0]


def fill_but(room):
    """Tensors that leave the device `room` bytes: all it gives (its runtime
    hands memory back that it had kept) beside a tensor of that size."""
    import torch
    kept, full, size = torch.empty(room, dtype=torch.uint8, device="cuda"), [], free()
    while size >= 4 << 20:
        try:
            full.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            size //= 2
    del kept
    torch.cuda.empty_cache()
    return full


def field(shape, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.rand(shape, generator=g, device="cuda", dtype=torch.float64) * 2.0 - 1.0


@pytest.mark.parametrize("par", [dict(), dict(precision=1), dict(krylov=1)])
def test_without_room_for_second_arrays(bx, par):
    import torch
    second = (N + 3) // 2 * (N + 2) ** 2 * 2 * (4 if par.get("precision") else 8)
    ba = bx.BoxArray.chop((0, 0, 0), (N - 1,) * 3, N)
    out, room = [], None
    for last in (False, False, True):
        ctx = bx.Context(0)
        phi = bx.MultiFab(ba, ctx=ctx).set_val(0.0)
        rhs = bx.MultiFab(ba, ctx=ctx).set_val(0.0).from_tensor(field((N,) * 3, 95))
        was = free()
        full = fill_but(room) if last else None
        lib, chk = bx._lib.lib(), bx._lib.check
        chk(lib.bxmg_profile_stage(ctx._h, 0))
        print("solve", par, "with %.0f MB" % (room / 1e6) if last else "with room", flush=True)
        res = bx.mlmg_solve(phi, rhs, fixed_cycles=3, **par)
        n, ms = C.c_int64(), C.c_double()
        chk(lib.bxmg_profile_read(ctx._h, C.byref(n), C.byref(ms), 1))
        room = was - free() - second // 2
        out.append((phi.slab.clone() if not last else phi.slab, n.value, res))
        del full
    _, (a, na, ra), (b, nb, rb) = out
    assert ra.cycles == rb.cycles == 3 and nb == 4 * na  # two launches a cycle, or one per half-sweep
    if par.get("krylov"):
        assert (a - b).abs().max() <= 1e-12 * a.abs().max()
    else:
        assert ra.hist == rb.hist and torch.equal(a, b)


def test_nodal_without_room_for_second_arrays(bx):
    ba = bx.BoxArray.chop((0, 0, 0), (N - 1,) * 3, N)
    second = (N + 2) // 2 * (N + 1) ** 2 * 16
    rhs = field((N + 1,) * 3, 96)
    phi = rhs.new_zeros(rhs.shape)
    out, room = [], None
    for dx in (0.5 / N, 1.0 / N, 2.0 / N):  # another cell width: another hierarchy, the solution times 4
        was = free()
        last = len(out) == 2
        full = fill_but(room) if last else None
        phi.zero_()
        print("nodal solve", "with %.0f MB" % (room / 1e6) if last else "with room", flush=True)
        res = bx.nodal_solve(ba, phi, rhs, fixed_cycles=3, dx=dx)
        room = was - free() - second // 2
        out.append((phi.cpu(), res))
        del full
    _, (a, ra), (b, rb) = out
    assert (4.0 * a - b).abs().max() <= 1e-12 * b.abs().max()
    assert max(abs(x - y) for x, y in zip(ra.hist, rb.hist)) <= 1e-12
