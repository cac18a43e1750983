"""Moments and columns on both sides of the size at which read-outs leave the
context's pinned memory (needs an MI355X): 2 MB is 87,381 nodes of three FP64
fields, 262,144 of one column.  Both ways give the sums of the populations, which
are read another way.
"""
from concurrent.futures import ThreadPoolExecutor

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


def test_buffers_pass_between_contexts_and_threads():
    """More contexts at once than buffers are kept, then new ones that take over the kept buffers, from
    several threads: each reads its own state."""
    def contexts(seed):
        runs = []
        for i in range(3):
            r = WL.paper_wave_run(0.0, L=16)
            r.nx, r.ny, r.rho = 7 + i, 20, np.random.default_rng(10 * seed + i).uniform(0.9, 1.1, (20, 7 + i))
            runs.append(r)
        for _ in range(3):
            L = [lbm.Lattice([r], precision="fp64") for r in runs]
            for k in L:
                k.init_all()
            for _ in range(2):
                for k, r in zip(L, runs):
                    # FP64 sums of nine numbers whose sum is the given density
                    assert np.max(np.abs(k.moments(0)[0] - r.rho)) <= 18 * 2.3e-16 * np.max(r.rho)
            for k in L:
                k.close()
        return True

    with ThreadPoolExecutor(3) as pool:
        assert all(pool.map(contexts, range(3)))
