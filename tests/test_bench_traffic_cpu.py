"""Counted HBM traffic is used only for the code it was taken on (CPU only): the
kernel's source file and the headers that hold its arithmetic, geometry and
memory access.  Every committed summary names both digests."""
import hashlib
import json
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1306_6445_amd", "csrc")


@pytest.fixture
def bench_module(tmp_path, monkeypatch):
    sys.path.insert(0, ROOT)
    import bench
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "traffic_%s_%s_%s.json"))
    return bench, tmp_path


def write(tmp, kernel, src, headers):
    with open(tmp / ("traffic_%s_fp32_config2.json" % kernel), "w") as fh:
        sha = hashlib.sha256(open(os.path.join(CSRC, src), "rb").read()).hexdigest()
        json.dump({"kernel_source_sha256": sha, "headers_sha256": headers, "nodes": 100, "bytes_per_dispatch": 7.0}, fh)


def test_a_changed_header_makes_counters_stale(bench_module, monkeypatch):
    bench, tmp = bench_module
    write(tmp, "multi", "lbm_multi.hip", bench.headers_sha256())
    assert bench.traffic_from_profile(100, "multi", "config2") == 7.0
    changed = tmp / "lbm_node.hpp"
    changed.write_text("// other arithmetic\n")
    monkeypatch.setattr(bench, "KERNEL_HEADERS", [str(changed) if h.endswith("lbm_node.hpp") else h
                                                  for h in bench.KERNEL_HEADERS])
    assert bench.traffic_from_profile(100, "multi", "config2") is None


def test_collide_counters_follow_the_single_step_source(bench_module):
    bench, tmp = bench_module
    write(tmp, "collide", "lbm_kernels.hip", bench.headers_sha256())
    assert bench.traffic_from_profile(100, "collide", "config2") == 7.0
    write(tmp, "collide", "lbm_multi.hip", bench.headers_sha256())
    assert bench.traffic_from_profile(100, "collide", "config2") is None


def test_every_header_of_the_step_kernels_is_hashed():
    sys.path.insert(0, ROOT)
    import bench
    hashed = {os.path.basename(h) for h in bench.KERNEL_HEADERS}
    todo = ["lbm_multi.hip", "lbm_kernels.hip", "lbm3d_kernels.hip", "lbm_mc_kernels.hip"]
    seen = set()
    while todo:
        for name in re.findall(r'#include "([^"/]+\.hpp)"', open(os.path.join(CSRC, todo.pop())).read()):
            if name not in seen:
                seen.add(name)
                todo.append(name)
    assert seen == hashed


def test_committed_summaries_name_both_digests():
    names = [n for n in os.listdir(os.path.join(ROOT, "profiles")) if n.startswith("traffic_") and n.endswith(".json")]
    assert names
    for name in names:
        with open(os.path.join(ROOT, "profiles", name)) as fh:
            t = json.load(fh)
        assert len(t["kernel_source_sha256"]) == 64 and len(t["headers_sha256"]) == 64, name
