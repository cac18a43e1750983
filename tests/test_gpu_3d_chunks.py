"""The fused 3D step against the two passes, bit for bit (needs an MI355X), at
the edges of its tiles and z chunks: grids narrower than a tile, one short of
and one past one, chunks of one plane to more than the grid, walls on every
axis and periodic seams (the paths with and without per-lane wall selects),
and the default schedule of a grid past the two-pass sizes.
"""
import dataclasses

import numpy as np
import pytest

from paper_1306_6445_amd import lbm, workloads as WL

pytestmark = pytest.mark.gpu


def run3(nx, ny, nz, walls=(0, 0, 0)):
    rng = np.random.default_rng(nx + 1000 * ny + nz)
    r = WL.droplet3_run(4, 1.0, 0.7, 0.4)
    z, y, x = np.mgrid[0:nz, 0:ny, 0:nx]
    shape = 0.5 + 0.5 * np.cos(2 * np.pi * x / nx) * np.cos(2 * np.pi * y / ny + 1) * np.cos(2 * np.pi * z / nz + 2)
    rho = (0.02 + 0.38 * shape) * (1 + 0.01 * rng.uniform(-1, 1, shape.shape))
    u = 0.02 * rng.uniform(-1, 1, (3,) + shape.shape)
    return dataclasses.replace(r, nx=nx, ny=ny, nz=nz, rho=rho, ux=u[0], uy=u[1], uz=u[2], bc_x=walls[0],
                               bc_y=walls[1], bc_z=walls[2])


def states(run, precision, schedule, steps=3):
    with lbm.Lattice3(run, precision=precision) as L:
        if schedule:
            L.set_schedule(*schedule)
        L.init_all()
        L.step(steps)
        return L.populations()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("walls", [(0, 0, 0), (1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1)])
@pytest.mark.parametrize("shape", [(1, 2, 1), (5, 7, 3), (31, 9, 6), (64, 8, 5), (65, 17, 12), (70, 33, 9)])
def test_tiles_and_chunks(shape, walls, precision):
    run = run3(*shape, walls)
    want = states(run, precision, (0, 64, 8, 64))
    for tile in ((64, 8), (32, 16), (32, 8), (64, 4), (64, 16)):
        for chunk in (1, 4, shape[2] + 5):
            assert np.array_equal(states(run, precision, (1,) + tile + (chunk,)), want), (tile, chunk)


@pytest.mark.parametrize("precision,shape", [("fp64", (96, 96, 40)), ("fp32", (96, 80, 40)), ("fp32", (150, 170, 150))])
def test_default_schedule(precision, shape):
    """150 x 170 x 150 FP32 populations outgrow the Infinity Cache (non-temporal stores)."""
    run = run3(*shape)
    assert np.array_equal(states(run, precision, None, 5), states(run, precision, (0, 64, 8, 64), 5))
