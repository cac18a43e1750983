"""Host-side checks of the kernels that advance several steps in one launch
(CPU only): tests/multi_maps_check.hip includes the same header functions the
library uses, is compiled for the host only and names what it checks.
"""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_multi_step_maps(tmp_path):
    exe = str(tmp_path / "multi_maps_check")
    subprocess.run([HIPCC, "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17",
                    "-I", os.path.join(ROOT, "include"), "-o", exe, os.path.join(ROOT, "tests", "multi_maps_check.hip")],
                   check=True, capture_output=True, text=True, timeout=600)
    p = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.startswith("ok"), p.stdout + p.stderr
