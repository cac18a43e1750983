"""The 3D fused step keeps its registers (CPU only): compiled for gfx950 with the
library's flags, no instance of it has scratch memory.  The populations that wait
for their collision sit in LDS; in registers they spilled.  FP64 with 64 x 16
tiles (1,024 threads of 128 registers, which a default schedule never takes)
cannot hold 19 doubles twice: it may not need more than the 348 bytes (444 with
64-bit addresses) of the kernel that kept them there without loads ahead; FP32
with that tile and 64-bit addresses not more than its 128.
"""
import os
import re
import subprocess

import pytest

from paper_1306_6445_amd import build as B

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1306_6445_amd", "csrc")


def scratch_bytes(src):
    """{kernel: scratch bytes per lane} from the compiler's resource remarks."""
    flags = [f for f in B.FLAGS if f not in ("-shared", "-fPIC") and not f.startswith(("-L", "-l"))]
    err = subprocess.run([B.HIPCC] + flags + ["--cuda-device-only", "-S", "-Rpass-analysis=kernel-resource-usage",
                                              "-o", os.devnull, os.path.join(CSRC, src)],
                         check=True, capture_output=True, text=True, timeout=900).stderr
    out, name = {}, None
    for line in err.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        name = m.group(1) if m else name
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m:
            out[name] = int(m.group(1))
    return out


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")
def test_fused_3d_step_does_not_spill():
    seen = 0
    for name, scratch in scratch_bytes("lbm3d_kernels.hip").items():
        m = re.search(r"fused3_kernelI([df])Li(\d+)ELi(\d+)ELb(\d)", name)
        if not m:
            continue
        seen += 1
        limit = 0
        if m.groups()[:3] == ("d", "64", "16"):
            limit = 348 if m.group(4) == "1" else 444
        elif m.groups() == ("f", "64", "16", "0"):
            limit = 128  # 64-bit addresses, past 4 GiB
        assert scratch <= limit, (name, scratch)
    assert seen == 30
