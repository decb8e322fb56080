"""Which workgroup takes what: the all-gather's numbering on the host, and launches at the sizes where it and the form
of the bf16 reduce-scatter change, against the oracle."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_all_gather_order(tmp_path):
    exe = str(tmp_path / "all_gather_order")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2302_12445_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "all_gather_order.cpp"), "-o", exe], check=True)
    assert "all_gather_order: ok" in subprocess.run([exe], check=True, capture_output=True, text=True).stdout


def list_of_tiles(tiles, P, g):
    """Two tensors whose plan has that many tiles in all."""
    import paper_2302_12445_amd as dear
    import workloads as W
    for n in range(1, tiles * 4096, 509):
        sizes = [n + max(0, tiles - 8) * 4096, 9]
        if len(dear.dear_plan_tiles(dear.dear_plan(sizes, P, W.NO_LIMIT, g))[0]) == tiles:
            return sizes
    raise AssertionError(tiles)


# last chunks of 4 and of 0 (mod 8) parts, one chunk exactly, one tile more, half tiles (bf16 up to 160 and 1024) and whole ones
@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("tiles", [5, 6, 7, 160, 161, 1023, 1024, 1025])
def test_launches_around_the_limits(dtype, tiles):
    from test_gpu_parity import Pair, say, small_workload
    import workloads as W
    say("case: %d tiles, %s" % (tiles, dtype))
    pair = Pair(small_workload(list_of_tiles(tiles, 3, 2 if dtype == "bf16" else 4), 3, W.NO_LIMIT, dtype))
    for route, fused in (("calls", False), ("calls", True), ("iteration", False), ("iteration", True)):
        pair.run(iterations=1, route=route, fused=fused)
    pair.close()
