"""Several two-component steps in one launch against one step per launch, bit
for bit (needs an MI355X): grids smaller than a tile's margin, one short of and
one past a tile and several tiles of each variant (four steps of 8 x 8 nodes;
two of 28 x 12, 32 x 8 and 32 x 24), walls on either axis, step counts
that leave remainders, graphs that end on either buffer.

One step at a time is lbm_mc_step(1), which always takes the single-step kernel.
"""
import dataclasses

import numpy as np
import pytest

from paper_1306_6445_amd import lbm, workloads as WL

pytestmark = pytest.mark.gpu


def run(nx, ny, bcx=0, bcy=0):
    rng = np.random.default_rng(nx + 1000 * ny)
    r = WL.mc_drop_run(8, 2.0, 0.5)
    y, x = np.mgrid[0:ny, 0:nx]
    p = 0.5 + 0.5 * np.cos(2 * np.pi * (x / nx + 0.3)) * np.cos(2 * np.pi * (y / ny + 0.1))
    rho = [(0.05 + 0.9 * v) * (1 + 0.01 * rng.uniform(-1, 1, (ny, nx))) for v in (p, 1 - p)]
    u = 0.02 * rng.uniform(-1, 1, (2, ny, nx))
    return dataclasses.replace(r, nx=nx, ny=ny, bc_x=bcx, bc_y=bcy, rhoA=rho[0], rhoB=rho[1], ux=u[0], uy=u[1])


def same(r, precision, steps, graph_steps=None):
    with lbm.LatticeMC(r, precision=precision) as L, lbm.LatticeMC(r, precision=precision) as S:
        if graph_steps is not None:
            L.set_graph_steps(graph_steps)
        L.init_all()
        S.init_all()
        for n in steps:
            L.step(n)
            for _ in range(n):
                S.step(1)
            assert np.array_equal(L.populations(), S.populations()), (n, r.nx, r.ny)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("walls", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("shape", [(1, 1), (2, 3), (7, 9), (16, 17), (100, 61), (170, 140), (448, 401), (833, 900),
                                   (607, 721), (960, 960)])
def test_grids(shape, walls, precision):
    same(run(*shape, *walls), precision, [4, 7, 2, 1])


@pytest.mark.parametrize("graph_steps", [1, 3, 8])
def test_graphs_from_either_buffer(graph_steps):
    same(run(90, 70, 0, 1), "fp32", [17, 1, 32, 5], graph_steps)
