"""The nodal solver's streaming smoother and one-workgroup coarse levels at
the sizes where they change shape: levels of one block, blocks that do not
divide the level or span it in one direction only, the smallest levels, all
mixes of boundaries.  Fixed-cycle iterates equal the oracle's to 1e-12
relative (the same stages in the same order; only the bottom CG sums in
another), and a solve from a nonzero guess over nonzero boundary values keeps
those and meets its tolerance by the oracle's operator.
"""
import numpy as np
import pytest

import workloads as W
from test_gpu_nodal import bx, dev, host, nodes, unknown_mask  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,per", [
    ((4, 4, 4), (0, 0, 0)),
    ((8, 4, 12), (1, 0, 1)),
    ((16, 16, 16), (1, 1, 1)),
    ((16, 160, 24), (0, 1, 0)),
    ((208, 16, 32), (1, 0, 0)),
    ((32, 24, 176), (0, 0, 1)),
    ((96, 112, 80), (0, 0, 0)),
    ((112, 72, 96), (1, 1, 1)),
])
def test_nodal_streamed_levels(bx, orc, n, per):  # noqa: F811
    bc = tuple(bx.PERIODIC if p else bx.DIRICHLET0 for p in per)
    ba = bx.BoxArray.chop((0, 0, 0), tuple(x - 1 for x in n), 32, bc=bc)
    m = unknown_mask(n, per)
    f = np.asfortranarray(W.uniform_rhs(nodes(n), 65))
    if per == (1, 1, 1):
        f = np.asfortranarray(f - f[m].mean())
    phi, rhs = dev(np.zeros(nodes(n))), dev(f)
    res = bx.nodal_solve(ba, phi, rhs, fixed_cycles=2)
    uo, io = orc.nodal_solve(n, per, f, fixed_cycles=2)
    assert res.cycles == 2 and res.levels == io["levels"]
    assert np.max(np.abs(host(phi) - uo)) <= 1e-12 * np.max(np.abs(uo))
    if any(per):
        return
    g = W.uniform_rhs(nodes(n), 66)
    phi = dev(g)
    res = bx.nodal_solve(ba, phi, rhs)
    u = host(phi)
    assert res.ok and np.array_equal(u[~m], g[~m])
    r = (f - orc.nodal_apply(n, per, 1.0 / n[0], u))[m]
    assert np.max(np.abs(r)) <= 1e-10 * np.max(np.abs(f[m]))
