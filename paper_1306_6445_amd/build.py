"""Builds the HIP library liblbm_mi355x.so in-tree for gfx950 with hipcc.

Usage:  python -m paper_1306_6445_amd.build
"""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "liblbm_mi355x.so")
SOURCES = [os.path.join(HERE, "csrc", n) for n in ("lbm_api.hip", "lbm_kernels.hip", "lbm_multi.hip", "mlp_api.hip", "mlp_kernels.hip",
                                                    "lbm3d_api.hip", "lbm3d_kernels.hip", "lbm_mc_api.hip",
                                                    "lbm_mc_kernels.hip")]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed FP32 instructions are kept out of every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # multiply-add contraction only within one source expression (HIP's
    # default also fuses across statements, depending on the surrounding
    # code), so that kernels sharing a device function round alike and the
    # fused and two-kernel schedules give the same bits
    "-ffp-contract=on",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"),
    # roctx ranges around the public calls (resolved through the ROCm runpath)
    "-L/opt/rocm/lib", "-lrocprofiler-sdk-roctx",
]


def build(verbose: bool = True) -> str:
    """Compiles every source to an object in parallel (each translation unit
    launches only its own kernels, so no device link step is needed), then
    links the shared library."""
    import concurrent.futures
    import tempfile

    tmp = LIB + ".tmp%d" % os.getpid()
    compile_flags = [f for f in FLAGS if f != "-shared" and not f.startswith("-L") and not f.startswith("-l")]
    link_flags = ["--offload-arch=gfx950", "-shared", "-fPIC"] + [f for f in FLAGS if f.startswith("-L") or f.startswith("-l")]
    jobs = max(1, min(len(SOURCES), int(os.environ.get("MAX_JOBS", os.cpu_count() or 1)), 16))
    with tempfile.TemporaryDirectory(prefix="lbm_build_") as d:
        objs = [os.path.join(d, os.path.basename(src) + ".o") for src in SOURCES]
        cmds = [[HIPCC] + compile_flags + ["-c", "-o", o, src] for src, o in zip(SOURCES, objs)]
        if verbose:
            for c in cmds:
                print(" ".join(c), flush=True)
        with concurrent.futures.ThreadPoolExecutor(jobs) as pool:
            for f in [pool.submit(subprocess.check_call, c) for c in cmds]:
                f.result()
        link = [HIPCC] + link_flags + ["-o", tmp] + objs
        if verbose:
            print(" ".join(link), flush=True)
        subprocess.check_call(link)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-q" not in sys.argv)
