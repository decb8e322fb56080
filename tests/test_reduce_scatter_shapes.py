"""The reduce-scatter in each depth, with and without a rest of replicas, in parts and in whole tiles, on both sides of the lines between
them, and the update on both sides of its line, against the oracle (the same bits)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _shapes_program(tmp_path):
    exe = str(tmp_path / "reduce_scatter_shapes")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2302_12445_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "reduce_scatter_shapes.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_rows_and_shapes_on_the_host(tmp_path):
    assert "reduce_scatter_shapes: ok" in subprocess.run([_shapes_program(tmp_path)], check=True, capture_output=True, text=True).stdout


def full(tiles):
    return [tiles * 4096 - 4099, 3]


SHORT = [900, 3, 911, 1]  # per tensor and shard far less than a tile
SOME = (SHORT * 60 + [16_400] + SHORT * 60) * 4  # and a few whole tiles among them, in a launch long enough for it
ODD = [4101, 9_003, 6_555]  # most tiles begin or end inside a vector

# replicas a lane: 1; 2 alone, with batches, with a rest; 4; 8; then rows (512 items and some behind them); whole tiles; very long launches
CASES = [("f32", 1, full(1030)), ("f32", 2, full(40)), ("f32", 3, full(321)), ("f32", 4, full(30)), ("f32", 6, full(200)), ("f32", 7, full(60)),
         ("f32", 8, full(20)), ("f32", 9, full(30)), ("f32", 16, full(63)), ("f32", 12, full(100)), ("f32", 13, full(127)), ("f32", 8, full(520)),
         ("f32", 9, full(330)), ("f32", 41, full(260)), ("f32", 3, SHORT * 100), ("f32", 8, SHORT * 30), ("f32", 9, SHORT * 30), ("f32", 16, SHORT * 20),
         ("f32", 5, SHORT * 80), ("f32", 7, full(2060)), ("f32", 8, full(6010)), ("f32", 5, full(6010)), ("f32", 4, full(6010)),
         ("bf16", 1, full(600)), ("bf16", 2, full(520)), ("bf16", 3, full(100)), ("bf16", 4, full(200)), ("bf16", 5, full(1030)), ("bf16", 6, full(100)),
         ("bf16", 8, full(100)), ("bf16", 9, full(12)), ("bf16", 4, full(60)), ("bf16", 8, full(130)), ("bf16", 7, full(45)), ("f32", 4, full(80)), ("f32", 12, full(365)), ("bf16", 24, full(515)), ("bf16", 6, full(1605)), ("f32", 6, full(80)), ("bf16", 16, full(200)), ("bf16", 13, full(250)), ("bf16", 9, full(600)), ("bf16", 8, full(2060)),
         ("bf16", 24, full(1030)), ("bf16", 2, SHORT * 200), ("bf16", 8, SHORT * 30), ("bf16", 11, SHORT * 30), ("bf16", 3, SHORT * 120),
         # the forms that are left, and whole tiles among short ones
         ("f32", 1, ODD * 3), ("f32", 2, ODD * 3), ("f32", 16, full(40)), ("bf16", 1, ODD * 3), ("bf16", 2, ODD * 3), ("bf16", 16, full(40)),
         ("f32", 1, SHORT * 150), ("f32", 2, SHORT * 150), ("f32", 4, SHORT * 100), ("f32", 8, SHORT * 80), ("bf16", 1, SHORT * 200),
         ("bf16", 8, SHORT * 200), ("bf16", 11, SHORT * 250), ("f32", 2, SOME), ("f32", 3, SOME), ("f32", 8, SOME), ("f32", 9, SOME),
         ("bf16", 2, SOME), ("bf16", 3, SOME), ("bf16", 8, SOME), ("bf16", 9, SOME), ("bf16", 4, SHORT * 200), ("bf16", 5, SHORT * 200),
         # weights of some parts with short vectors between them: in parts, then so many that tiles go whole
         ("f32", 8, [2900, 33, 900] * 60), ("bf16", 16, [2900, 33, 900] * 90), ("f32", 3, ([2900] + [33, 900] * 6) * 90),
         ("bf16", 5, ([3900] + [33, 900] * 8) * 50)]


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_the_cases_reach_every_form(tmp_path):
    """Which kernels the cases below launch, by the library's own rule: each depth and rest in parts and in whole tiles, both types, the
    batch kernel, and whole tiles among short ones in the form that takes tiles whole."""
    import paper_2302_12445_amd as dear
    asked, of = [], []
    for dtype, P, sizes in CASES:
        g = 4 if dtype == "f32" else 2
        v = 16 // g
        tiles = dear.dear_plan_tiles(dear.dear_plan(sizes, P, dear.DEAR_NO_LIMIT, g))[0]
        runs = [t for t in tiles if t.layer >= 0]
        whole = sum(t.count == 4096 for t in runs)
        several = sum((t.src_begin + t.count - 1) // v - t.src_begin // v >= 256 for t in runs)  # parts
        cut = sum(t.src_begin % v != 0 or (t.src_begin + t.count) % v != 0 for t in runs)
        for updates in (0, 1):
            asked.append("%d %d 0 %d %d %d %d %d\n" % (g == 2, updates, P, sum(t.count for t in runs), len(tiles), several, cut))
            of.append((dtype, P, whole))
    said = subprocess.run([_shapes_program(tmp_path), "ask"], input="".join(asked), check=True, capture_output=True, text=True).stdout.splitlines()
    reached, whole_among_short = set(), set()
    for (dtype, P, whole), line in zip(of, said):
        depth, _, _, in_tiles = map(int, line.split())
        rest = "batch kernel" if depth == 0 else "none" if P == depth and not in_tiles else "batches" if P % depth == 0 else "tail"
        reached.add((dtype, depth, rest, bool(in_tiles)))
        if in_tiles and whole:
            whole_among_short.add((dtype, P % depth == 0))
    for dtype in ("f32", "bf16"):
        forms = [(0, "batch kernel", False), (1, "none", False), (1, "batches", True)]
        forms += [(d, rest, False) for d in (2, 4, 8) for rest in ("none", "batches", "tail")]
        forms += [(d, rest, True) for d in (2, 4, 8) for rest in ("batches", "tail")]
        assert {(dtype,) + f for f in forms} == {r for r in reached if r[0] == dtype}
    assert whole_among_short == {("f32", True), ("f32", False), ("bf16", True), ("bf16", False)}


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
