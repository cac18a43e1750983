"""Population buffers between 2 and 4 GiB (needs an MI355X), whose byte offsets set
the top bit of the 32-bit ones that the several-step kernels and the fused 3D step
use, with walls, whose slots are selected per lane; and the sizes just below and
past 4 GiB, where several steps a launch end.  Bit for bit against single steps
(two passes in 3D): equal densities and velocities at every node after a last
step of the same kind."""
import dataclasses

import numpy as np
import pytest

from paper_1306_6445_amd import lbm, workloads as WL
from tests.test_gpu_3d_chunks import run3
from tests.test_gpu_mc_multi_step import run as run_mc
from tests.test_gpu_multi_step import run

pytestmark = pytest.mark.gpu

GIB = 2 ** 30


def fields(L, calls, several):
    L.init_all()
    for n in calls:
        L.step(n)
    assert several is None or (L.steps_per_launch > 1) == several
    return L.moments()


def same(a, b):
    for u, v in zip(a, b):
        assert np.array_equal(u, v)


@pytest.mark.parametrize("precision,size,shape", [("fp32", 4, (10880, 10900)), ("fp64", 8, (7700, 7700)),
                                                  ("bf16", 2, (11000, 11000))])
def test_one_component(precision, size, shape):
    assert 2 * GIB < 9 * size * shape[0] * shape[1] < 4 * GIB
    r = run(*shape, 1, 1)
    got = []
    for calls, fused in (([1] * 4 + [2], 2), ([4, 2], 2), ([6], 0)):
        with lbm.Lattice([r], precision=precision, fused=fused) as L:
            got.append(fields(L, calls, fused > 0))
    same(got[0], got[1])
    same(got[0], got[2])


@pytest.mark.parametrize("precision,size,below,past", [("fp32", 4, (10880, 10900), (10880, 11000)),
                                                       ("fp64", 8, (7700, 7700), (7750, 7750)),
                                                       ("bf16", 2, (15400, 15400), (15500, 15500))])
def test_several_steps_end_at_4_gib(precision, size, below, past):
    small = run(8, 8)
    for shape, several in ((below, True), (past, False)):
        assert (9 * size * shape[0] * shape[1] < 4 * GIB) == several
        with lbm.Lattice([dataclasses.replace(small, nx=shape[0], ny=shape[1])], precision=precision) as L:
            assert (L.steps_per_launch > 1) == several


@pytest.mark.parametrize("precision,size,n", [("fp32", 4, 7700), ("fp64", 8, 5440)])
def test_two_components(precision, size, n):
    assert 2 * GIB < 18 * size * n * n < 4 * GIB
    with lbm.LatticeMC(run_mc(n, n, 1, 1), precision=precision) as L:
        want = fields(L, [1] * 4 + [2], True)
        same(want, fields(L, [4, 2], True))


@pytest.mark.parametrize("precision,size,n", [("fp32", 4, 380), ("fp64", 8, 300)])
def test_three_dimensions(precision, size, n):
    assert 2 * GIB < 19 * size * n ** 3 < 4 * GIB
    with lbm.Lattice3(run3(n, n, n, (1, 1, 1)), precision=precision) as L:
        got = fields(L, [3], None)
        L.set_schedule(0)
        same(got, fields(L, [3], None))
