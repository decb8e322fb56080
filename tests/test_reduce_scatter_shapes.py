"""The reduce-scatter in each depth, with and without a rest of replicas, in parts and in whole tiles, on both sides of the lines between
them, and the update on both sides of its line, against the oracle (the same bits)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_rows_and_shapes_on_the_host(tmp_path):
    exe = str(tmp_path / "reduce_scatter_shapes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2302_12445_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "reduce_scatter_shapes.cpp"), "-o", exe], check=True)
    assert "reduce_scatter_shapes: ok" in subprocess.run([exe], check=True, capture_output=True, text=True).stdout


def full(tiles):
    return [tiles * 4096 - 4099, 3]


SHORT = [900, 3, 911, 1]  # per tensor and shard far less than a tile

# replicas a lane: 1; 2 alone, with batches, with a rest; 4; 8; then rows (512 items and some behind them); whole tiles; very long launches
CASES = [("f32", 1, full(1030)), ("f32", 2, full(40)), ("f32", 3, full(321)), ("f32", 4, full(30)), ("f32", 6, full(200)), ("f32", 7, full(60)),
         ("f32", 8, full(20)), ("f32", 9, full(30)), ("f32", 16, full(63)), ("f32", 12, full(100)), ("f32", 13, full(127)), ("f32", 8, full(520)),
         ("f32", 9, full(330)), ("f32", 41, full(260)), ("f32", 3, SHORT * 100), ("f32", 8, SHORT * 30), ("f32", 9, SHORT * 30), ("f32", 16, SHORT * 20),
         ("f32", 5, SHORT * 80), ("f32", 7, full(2060)), ("f32", 8, full(6010)), ("f32", 5, full(6010)), ("f32", 4, full(6010)),
         ("bf16", 1, full(600)), ("bf16", 2, full(520)), ("bf16", 3, full(100)), ("bf16", 4, full(200)), ("bf16", 5, full(1030)), ("bf16", 6, full(100)),
         ("bf16", 8, full(100)), ("bf16", 9, full(12)), ("bf16", 4, full(60)), ("bf16", 8, full(130)), ("bf16", 7, full(45)), ("f32", 4, full(80)), ("f32", 12, full(365)), ("bf16", 24, full(515)), ("bf16", 6, full(1605)), ("f32", 6, full(80)), ("bf16", 16, full(200)), ("bf16", 13, full(250)), ("bf16", 9, full(600)), ("bf16", 8, full(2060)),
         ("bf16", 24, full(1030)), ("bf16", 2, SHORT * 200), ("bf16", 8, SHORT * 30), ("bf16", 11, SHORT * 30), ("bf16", 3, SHORT * 120)]


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P,sizes", CASES)
def test_every_shape_gives_the_oracles_bits(dtype, P, sizes):
    import numpy as np
    import torch
    import paper_2302_12445_amd as dear
    import workloads as W
    from paper_2302_12445_amd import binding as B
    from test_gpu_parity import Pair, say, small_workload
    say("case: reduce-scatter shapes, %s, P=%d, %d tensors, %d elements" % (dtype, P, len(sizes), sum(sizes)))
    pair = Pair(small_workload(sizes, P, W.NO_LIMIT, dtype))
    n_tiles = len(dear.dear_plan_tiles(pair.em.plan)[0])
    for route, fused, width in (("calls", False, 0), ("calls", True, 0), ("iteration", False, 0), ("iteration", True, 0),
                                ("calls", True, n_tiles + 1)):  # a bound between the number of tiles and that of parts
        pair.run(iterations=1, route=route, fused=fused, width=width)
    if sum(sizes) < 4_000_000:
        em = pair.em
        em.shard_grad.fill_(float("nan"))
        dear.dear_reduce_scatter_static(em.plan, B.DEAR_F32 if dtype == "f32" else B.DEAR_BF16, [t.data_ptr() for rep in em.grads for t in rep],
                                        -1, em.shard_grad.data_ptr(), torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        pair.compare_buffer("shard_grad, static call", em.shard_grad, pair.sg)
    assert np.isfinite(pair.sg).any()
    pair.close()


@pytest.mark.gpu
@pytest.mark.parametrize("P,sizes,buckets", [(2, [11_990 * 1024], 1), (2, [12_300 * 1024 + 5], 1), (3, [12_100 * 1024 + 77] * 2, 2), (5, [11_000 * 1024, 12_289 * 1024], 2)])
def test_update_in_rows_gives_the_oracles_bits(P, sizes, buckets):
    import workloads as W
    from test_gpu_parity import Pair, say, small_workload
    say("case: update in rows, P=%d, %d buckets, %d elements" % (P, buckets, sum(sizes)))
    pair = Pair(small_workload(sizes, P, W.NO_LIMIT if buckets == 1 else max(sizes) * 4, "f32"))
    assert pair.em.plan.n_buckets == buckets
    for per_bucket in (True, False):
        pair.run(iterations=1, route="calls", per_bucket=per_bucket)
    pair.close()
