"""ParallelCopy of enough cells for several per thread, bitwise against the
oracle's: odd edges (blocks of cells that straddle regions, a partial last
block), ghosts, component ranges and both precisions."""
import pytest

import test_gpu_pcopy
from test_gpu_pcopy import bx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("dhi,per,mb_src,mb_dst,ng,ngc", [
    ((130, 128, 126), (1, 0, 1), 64, 48, 1, 1),
    ((150, 98, 142), (0, 0, 0), 37, 71, 2, 0),
])
def test_large_parallel_copy_bitwise(bx, orc, dhi, per, mb_src, mb_dst, ng, ngc, dtype):  # noqa: F811
    test_gpu_pcopy.test_parallel_copy_bitwise(bx, orc, (0, 0, 0), dhi, per, mb_src, mb_dst, ng, ngc, dtype)
