"""bench.py counts the steps of a launch as the library reports them (CPU only)."""
import os
import sys
from types import SimpleNamespace

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("prec,per_node", [("fp64", 144), ("fp32", 72), ("bf16", 44)])
@pytest.mark.parametrize("steps", [1, 2, 4])
def test_a_fused_launch_moves_the_state_once_in_its_steps(prec, per_node, steps):
    sys.path.insert(0, ROOT)
    import bench
    # 1000 steps of 5 us: a launch takes steps x 5 us and moves the populations once each way
    ms, rate = bench.step_kernel(SimpleNamespace(steps_per_launch=steps), 2, prec, 65536, 5e-3, 1000, None)
    assert ms == pytest.approx(5e-3 * steps)
    assert rate == pytest.approx(per_node * 65536 / (5e-6 * steps) / 1e9)


def test_the_two_kernel_schedule_counts_its_collide_launch():
    sys.path.insert(0, ROOT)
    import bench
    ms, rate = bench.step_kernel(SimpleNamespace(steps_per_launch=1), 0, "fp32", 65536, 5e-3, 1000, 0.003)
    assert ms == pytest.approx(0.003) and rate == pytest.approx(76 * 65536 / 3e-6 / 1e9)
