"""Moments and columns on both sides of the size at which read-outs leave the
context's pinned memory (needs an MI355X): 2 MB is 87,381 nodes of three FP64
fields, 262,144 of one column.  Both ways give the sums of the populations, which
are read another way.
"""
import numpy as np
import pytest

from paper_1306_6445_amd import lbm, workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(1, 1), (3, 29127), (3, 29128), (291, 301), (2, 262144), (2, 262145)])
def test_moments_and_columns(shape, precision):
    nx, ny = shape
    r = WL.paper_wave_run(0.0, L=16)
    r.nx, r.ny, r.rho = nx, ny, np.random.default_rng(ny).uniform(0.9, 1.1, (ny, nx))
    with lbm.Lattice([r, r], precision=precision) as L:
        L.init_all()
        L.step(3)
        for i in (1, 0):
            f = L.populations(i)
            rho, ux, uy = L.moments(i)
            # FP64 sums of the same nine numbers in another order
            assert np.max(np.abs(rho - f.sum(axis=0))) <= 9 * 2.3e-16 * np.max(rho)
            assert np.all(np.isfinite(ux)) and np.all(np.isfinite(uy))
            for x in (0, nx - 1):
                assert np.max(np.abs(L.density_column(i, x) - rho[:, x])) <= 9 * 2.3e-16 * np.max(rho)
