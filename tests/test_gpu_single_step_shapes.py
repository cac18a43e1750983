"""Every shape of the single fused step (needs an MI355X), asked for one step at a
time, so that each step of either parity is a launch of its own: interior,
periodic and wall tiles of the one-node halo against the two-kernel schedule, bit
for bit."""
import numpy as np
import pytest

from paper_1306_6445_amd import lbm, workloads as WL
from tests.helpers import small_run

pytestmark = pytest.mark.gpu

W = WL.BC_WALL


@pytest.mark.parametrize("prec", ["fp64", "fp32", "bf16"])
def test_single_steps_of_every_shape(prec):
    runs = [small_run(300, 200, "cs", kappa=0.6, bc_y=W, seed=31), small_run(257, 130, "pw", kappa=0.3, seed=32),
            small_run(200, 190, "exp", kappa=0.0, bc_x=W, bc_y=W, seed=33), small_run(20, 7, "cs", bc_x=W, seed=34)]

    def go(tile, fused, calls):
        with lbm.Lattice(runs, precision=prec, tile=tile, fused=fused) as L:
            L.init_all()
            for n in calls:
                L.step(n)
            return [L.populations(i) for i in range(len(runs))]

    ref = go((64, 4), 0, [5])
    for tile in ((64, 4), (32, 8), (128, 2), (256, 1), (256, 2), (128, 4), (64, 8), (64, 2)):
        for fused in (1, 2, 4):
            for u, v in zip(ref, go(tile, fused, [1] * 5)):
                np.testing.assert_array_equal(u, v, err_msg="%s %d" % (tile, fused))
