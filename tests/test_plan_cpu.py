"""The planner of the streaming sweeps runs on the host in the first solve of a
geometry, so its search has to be short: under 5 ms for a level-0 plan of large
levels (0.1 here; pricing every number of pieces instead of every size of a
piece took 8 to 22, three plans a hierarchy).  And its blocks cover the level.
"""
import ctypes as C
import time

import pytest

I32 = C.c_int32


@pytest.fixture(scope="module")
def plan():
    import paper_2403_12179_amd as bx
    fn = bx._lib.lib()["_ZN4bxmg10plan_sweepEPKiS1_ibbiii"]  # bxmg::plan_sweep, its result through a pointer
    fn.restype = None

    def call(n, per, kind, zero, f32, mode):
        out = (I32 * 128)()
        fn(C.byref(out), (I32 * 3)(*n), (I32 * 3)(*per), I32(kind), C.c_bool(zero), C.c_bool(f32), I32(mode),
           I32(256), I32(1024))
        keys = ("nt threads blocks pad n0 n1 n2 p0 p1 p2 H GH cs RM RY hm hy XM TY ZC nbx nby nbz").split()
        return dict(zip(keys, out))
    return call


@pytest.mark.parametrize("n", [(1024, 1024, 64), (512, 512, 512), (2048, 256, 128), (256, 256, 256)])
@pytest.mark.parametrize("kind,f32,mode", [(0, False, 0), (2, False, 0), (0, True, 1)])
def test_search_time(plan, n, kind, f32, mode):
    best = 1e9
    for _ in range(5):
        t = time.perf_counter()
        P = plan(n, (0, 0, 1), kind, f32, f32, mode)
        best = min(best, time.perf_counter() - t)
    assert best < 5e-3
    assert (P["n0"], P["n1"], P["n2"], P["p2"]) == (*n, 1) and 0 < P["threads"] <= P["nt"] <= 1024
    assert P["RM"] * P["RY"] <= P["threads"] and P["blocks"] == P["nbx"] * P["nby"] * P["nbz"]
    for cells, own, blocks in ((n[0] // 2, P["XM"], P["nbx"]), (n[1], P["TY"], P["nby"]), (n[2], P["ZC"], P["nbz"])):
        assert own * blocks >= cells > own * (blocks - 1)
