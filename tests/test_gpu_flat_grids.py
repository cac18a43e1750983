"""Grids a few nodes high (needs an MI355X): many of them, or long ones, take single
steps, because tiles of several steps would do most of their work beyond the
grid; grids that fill the tiles and launches of few tiles keep several steps.  A
step of the flat grids takes no longer than one asked for by itself (lbm_step(1),
whose launch overhead is below the kernel's time there); 1.1 covers the spread of
repeated timings, several steps a launch took 1.3 to 1.5 times as long."""
import time

import pytest

from paper_1306_6445_amd import lbm
from tests.test_gpu_mc_multi_step import run as run_mc
from tests.test_gpu_multi_step import run

pytestmark = pytest.mark.gpu


def seconds(L, calls, n):
    best = float("inf")
    for _ in range(5):
        L.synchronize()
        t = time.perf_counter()
        for _ in range(calls):
            L.step(n)
        L.synchronize()
        best = min(best, time.perf_counter() - t)
    return best


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape,runs", [((1000000, 4), 1), ((256, 4), 2000), ((300000, 8), 1)])
def test_flat_grids_are_no_slower_than_single_steps(shape, runs, precision):
    r = run(*shape)
    with lbm.Lattice([r] * runs, precision=precision) as L:
        L.init_all()
        L.step(66)
        assert seconds(L, 1, 64) <= 1.1 * seconds(L, 64, 1)
        assert L.steps_per_launch == 1


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape,runs", [((60000, 20), 1), ((20000, 8), 1), ((64, 64), 100), ((20, 20), 300)])
def test_other_grids_keep_several_steps(shape, runs, precision):
    with lbm.Lattice([run(*shape)] * runs, precision=precision) as L:
        assert L.steps_per_launch > 1


@pytest.mark.parametrize("precision,shape", [("fp32", (400000, 4)), ("fp32", (200000, 8)), ("fp64", (1000000, 1))])
def test_flat_two_component_grids_are_no_slower_than_single_steps(precision, shape):
    with lbm.LatticeMC(run_mc(*shape), precision=precision) as L:
        L.init_all()
        L.step(66)
        assert seconds(L, 1, 64) <= 1.1 * seconds(L, 64, 1)
        assert L.steps_per_launch == 1


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(100000, 20), (4, 100000), (600, 600)])
def test_other_two_component_grids_keep_several_steps(shape, precision):
    with lbm.LatticeMC(run_mc(*shape), precision=precision) as L:
        assert L.steps_per_launch > 1
