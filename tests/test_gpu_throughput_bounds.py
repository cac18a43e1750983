"""Throughput of the default schedules above what one step a launch reaches (needs
an MI355X), so that losing the several-step kernels or the 3D schedules that fill
the CUs trips them.  Measured, MLUPS with them and without: the 40 x 256^2 FP32
sweep 103k / 79k (two kernels a step 52k), 256 slabs of 4 x 256 FP32 69k / 6.7k, one
100^2 FP64 run 4.2k / 1.6k, the 2048^2 mixture FP32 42k / 33k and FP64 21k / 17k, 160^3
FP32 28k / 13k, 96^3 FP64 14.6k / 1.7k.  Each bound lies between, nearer to the lower
figure where the two are far apart."""
import time

import pytest

from paper_1306_6445_amd import lbm, workloads as WL
from tests.test_gpu_multi_step import run

pytestmark = pytest.mark.gpu


def mlups(L, nodes, k):
    L.step(64)
    L.synchronize()
    best = 0.0
    for _ in range(5):
        t = time.perf_counter()
        L.step(k)
        L.synchronize()
        best = max(best, nodes * k / (time.perf_counter() - t) / 1e6)
    return best


def test_fp32_sweep():
    runs = WL.config2()
    nodes = sum(r.nodes for r in runs)
    with lbm.Lattice(runs, precision="fp32") as L:
        L.init_all()
        several = mlups(L, nodes, 2000)
        L.set_fused(0)
        two = mlups(L, nodes, 2000)
    assert several > 88000 and several > 1.65 * two


@pytest.mark.parametrize("precision,shape,runs,bound", [("fp32", (4, 256), 256, 35000), ("fp64", (100, 100), 1, 2700)])
def test_small_grids(precision, shape, runs, bound):
    with lbm.Lattice([run(*shape)] * runs, precision=precision) as L:
        L.init_all()
        assert mlups(L, shape[0] * shape[1] * runs, 1000) > bound


@pytest.mark.parametrize("precision,bound", [("fp32", 36500), ("fp64", 18700)])
def test_mixture(precision, bound):
    r = WL.mc_spinodal_run(2048)
    with lbm.LatticeMC(r, precision=precision) as L:
        L.init_all()
        assert mlups(L, r.nodes, 256) > bound


@pytest.mark.parametrize("precision,n,bound", [("fp32", 160, 20000), ("fp64", 96, 8000)])
def test_three_dimensions(precision, n, bound):
    r = WL.config3d(n)
    with lbm.Lattice3(r, precision=precision) as L:
        L.init_all()
        assert mlups(L, r.nodes, 96) > bound
