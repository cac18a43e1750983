"""Steps that a launch takes, as the library reports them (needs an MI355X): four
on grids of few tiles, two on others, one with the two-kernel
schedule or a multi-range run."""
import dataclasses

import pytest

from paper_1306_6445_amd import lbm
from tests.test_gpu_mc_multi_step import run as run_mc
from tests.test_gpu_multi_step import run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
def test_single_component(precision):
    for shape, n, want in (((100, 100), 1, 4), ((256, 256), 40, 2), ((4, 100), 20, 4)):
        with lbm.Lattice([dataclasses.replace(run(*shape), kappa=0.0)] * n, precision=precision) as L:
            assert L.steps_per_launch == want
            L.set_fused(0)
            assert L.steps_per_launch == 1
            L.set_fused(2)
            L.set_multirange(0, -1.0, 0.1)
            assert L.steps_per_launch == 1


def test_plain_fp64_run_of_256_squared_takes_four():
    with lbm.Lattice([run(256, 256)], precision="fp64") as L:
        assert L.steps_per_launch == 4


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_two_components(precision):
    for shape, want in (((100, 100), 4), ((900, 800), 2)):
        with lbm.LatticeMC(run_mc(*shape), precision=precision) as L:
            assert L.steps_per_launch == want
