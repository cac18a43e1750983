"""The kernels that advance several steps in one launch, and the two-component
step, run no binary64 arithmetic in FP32 and bf16 storage (CPU only): the same
check of the gfx950 assembly as for the single-step kernels, for every instance
of multi_kernel, strip_kernel, mc_multi_kernel and mc_fused_kernel."""
import os
import re

import pytest

from paper_1306_6445_amd import build as B
from tests.test_precision_isa_cpu import CSRC, kernels_asm

KERNELS = {"lbm_multi.hip": {"multi_kernel": {"f": 9, "NS_6bf16_tE": 8, "d": 7}, "strip_kernel": {"f": 2, "d": 2}},
           "lbm_mc_kernels.hip": {"mc_multi_kernel": {"f": 3, "d": 2}, "mc_fused_kernel": {"f": 6, "d": 6}}}


@pytest.mark.skipif(not os.path.exists(B.HIPCC), reason="hipcc not installed")
@pytest.mark.parametrize("src", sorted(KERNELS))
def test_no_fp64_instructions_below_fp64(src, tmp_path):
    seen, f64_in_fp64 = {k: {} for k in KERNELS[src]}, 0
    for name, ops in kernels_asm(os.path.join(CSRC, src), str(tmp_path / "k.s")).items():
        m = re.search(r"\d(%s)I(f|NS_6bf16_tE|d)" % "|".join(KERNELS[src]), name)
        if not m:
            continue
        kernel, storage = m.groups()
        seen[kernel][storage] = seen[kernel].get(storage, 0) + 1
        f64 = [op for op in ops if "_f64" in op]
        if storage == "d":
            f64_in_fp64 += len(f64)
        else:
            assert not f64, (name, sorted(set(f64)))
    for kernel, least in KERNELS[src].items():
        for storage, n in least.items():
            assert seen[kernel].get(storage, 0) >= n, (kernel, seen)
    assert f64_in_fp64 > 0
