"""Steps recorded by a stream capture of the caller's (needs an MI355X): an even
number of recorded steps leaves the state where the recording found it, so
every replay advances it by that many steps, also with eager steps between the
replays, in every storage and at grids of each multi-step shape (four steps a
launch, two, strips) and from either parity.  Bit for bit against the same
steps without a capture.
"""
import numpy as np
import pytest
import torch

from paper_1306_6445_amd import lbm
from tests.test_gpu_mc_multi_step import run as run_mc
from tests.test_gpu_multi_step import run

pytestmark = pytest.mark.gpu


def replayed(L, before, recorded):
    """Steps that the replays and the eager steps around them have taken."""
    L.step(before)
    L.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=L.stream):
        L.step(recorded)
    total = before
    for eager in (0, 2, 40, 6):
        with torch.cuda.stream(L.stream):
            graph.replay()
            graph.replay()
        L.step(eager)
        L.synchronize()
        total += 2 * recorded + eager
    return total


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16"])
@pytest.mark.parametrize("shape", [(4, 61), (100, 61), (300, 520)])
@pytest.mark.parametrize("before,recorded", [(0, 2), (33, 4), (70, 6), (1, 40)])
def test_replays_of_recorded_steps_advance(shape, precision, before, recorded):
    runs = [run(*shape, 0, 1)]
    with lbm.Lattice(runs, precision=precision) as L, lbm.Lattice(runs, precision=precision) as S:
        L.init_all()
        S.init_all()
        S.step(replayed(L, before, recorded))
        assert np.array_equal(L.populations(), S.populations())


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("shape", [(100, 61), (600, 500)])
@pytest.mark.parametrize("before,recorded", [(0, 2), (33, 4)])
def test_replays_of_recorded_two_component_steps_advance(shape, precision, before, recorded):
    r = run_mc(*shape, 0, 1)
    with lbm.LatticeMC(r, precision=precision) as L, lbm.LatticeMC(r, precision=precision) as S:
        L.init_all()
        S.init_all()
        S.step(replayed(L, before, recorded))
        assert np.array_equal(L.populations(), S.populations())
