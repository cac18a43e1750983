"""Several steps in one launch against one step per launch, bit for bit (needs
an MI355X).

The multi-step kernel runs the collision of the single-step kernels on the same
rounded states (bf16 storage: the same writer densities and rounding bits), so
every population is equal.  The grids sit at the edges of its
tiles: smaller than a tile's margin, one short of and one past a tile, several
tiles of each variant (four steps of 8 x 8, 12 x 12, 16 x 16 and 20 x 20
nodes; two of
28 x 12, 28 x 20, 32 x 16, 32 x 24, 64 x 16, 60 x 12, 60 x 20, 60 x 24, 4 x 60 and
8 x 60; strips of 4 x 52 and 8 x 50), walls on either axis, batches of
uneven runs; step counts leave remainders and start at odd counts.
"""
import dataclasses

import numpy as np
import pytest

from paper_1306_6445_amd import lbm, workloads as WL

pytestmark = pytest.mark.gpu


def run(nx, ny, bcx=0, bcy=0, eos="cs", seed=0):
    rng = np.random.default_rng(seed + 1000 * nx + ny)
    if eos == "cs":
        r = WL.droplet_run(8, 2.0, 0.7, 0.4, 1.93)
        lo, hi = 0.02, 0.4
    else:
        r = WL.paper_droplet_run("pw" if eos == "pw" else "exp", 0.4, n=8, R=2.0)
        lo, hi = (1.0, 90.0) if eos == "pw" else (80.0, 500.0)
    y, x = np.mgrid[0:ny, 0:nx]
    shape = 0.5 + 0.5 * np.cos(2 * np.pi * (x / nx + 0.3)) * np.cos(2 * np.pi * (y / ny + 0.1))
    rho = (lo + (hi - lo) * shape) * (1 + 0.01 * rng.uniform(-1, 1, (ny, nx)))
    u = 0.02 * rng.uniform(-1, 1, (2, ny, nx))
    return dataclasses.replace(r, nx=nx, ny=ny, rho=rho, ux=u[0], uy=u[1], bc_x=bcx, bc_y=bcy)


def states(runs, precision, fused, steps, graph_steps=None):
    with lbm.Lattice(runs, precision=precision, fused=fused, graph_steps=graph_steps) as L:
        L.init_all()
        out = []
        for n in steps:
            L.step(n)
            out.append([L.populations(i) for i in range(len(runs))])
        status = L.status()
    return out, status


def same(runs, precision, steps, graph_steps=None):
    a, sa = states(runs, precision, 2, steps, graph_steps)
    b, sb = states(runs, precision, 0, steps)
    assert np.array_equal(sa, sb)
    for n, x, y in zip(steps, a, b):
        for i, (f, g) in enumerate(zip(x, y)):
            assert np.array_equal(f, g), (n, i, runs[i].nx, runs[i].ny)


SMALL = [(1, 1), (2, 3), (5, 1), (7, 9), (8, 8), (16, 17), (33, 25), (100, 61)]
LARGE = [(240, 200), (257, 241), (640, 33), (1200, 500), (700, 641), (599, 601), (607, 623),
         (145, 133), (209, 225), (301, 281), (353, 337), (401, 399)]


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("walls", [(0, 0), (1, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("shape", SMALL + LARGE)
def test_single_runs(shape, walls, precision):
    same([run(*shape, *walls)], precision, [1, 4, 9, 2])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shapes", [[(9, 8), (64, 65), (20, 41)],
                                    [(256, 256)] * 20,
                                    [(4, 256)] * 150 + [(3, 61)],
                                    [(8, 181)] * 90 + [(7, 60), (5, 120)],
                                    [(61, 400), (60, 20), (300, 300), (121, 119), (480, 260)] * 3])
def test_batches(shapes, precision):
    runs = [run(nx, ny, (i // 2) % 2, i % 2, seed=i) for i, (nx, ny) in enumerate(shapes)]
    same(runs, precision, [2, 3, 4])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shapes", [[(1, 1)], [(1, 300)], [(4, 52)], [(8, 50)], [(6, 49)], [(5, 101)], [(2, 3)],
                                    [(4, 51), (3, 53), (1, 105), (2, 2)], [(8, 51), (4, 100), (7, 149), (1, 9)]])
def test_strips(shapes, precision):
    """Grids of at most 4 or 8 nodes along a periodic x, walls along y on every second run."""
    for first in (0, 1):
        runs = [run(nx, ny, 0, (i + first) % 2, seed=i) for i, (nx, ny) in enumerate(shapes)]
        same(runs, precision, [4, 8, 1, 9, 2])


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("eos", ["pw", "exp"])
def test_other_equations_of_state(eos, precision):
    same([run(50, 40, 0, 1, eos), run(23, 60, 0, 0, eos)], precision, [4, 3])


@pytest.mark.parametrize("graph_steps", [1, 3, 16])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
@pytest.mark.parametrize("shape", [(90, 70), (300, 520)])
def test_graphs_from_either_buffer(shape, precision, graph_steps):
    """Replays whose number of launches is odd end on the other buffer; single
    steps between the replays change parity and buffer."""
    same([run(*shape)], precision, [35, 1, 64, 7, 33], graph_steps)


def test_divergence_inside_a_launch_is_flagged():
    r = run(64, 64)
    r.rho[10, 10] = 0.995  # eta just below 1: the node leaves the EOS's domain within the first steps
    with lbm.Lattice([r, run(64, 64, seed=1)], precision="fp64") as L:
        L.init_all()
        L.step(200)
        assert list(L.status()) == [1, 0]
