"""The all-gather in which each XCD takes an eighth of a chunk, on both sides of its lines, with last chunks of every length, in
replicas that lie alike and in others, against the oracle (the same bits, and nothing around the tensors written)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_numbering_and_rule_on_the_host(tmp_path):
    exe = str(tmp_path / "all_gather_eighths")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2302_12445_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "all_gather_eighths.cpp"), os.path.join(ROOT, "paper_2302_12445_amd", "csrc", "plan.cpp"),
                    "-o", exe], check=True)
    assert "all_gather_eighths: ok" in subprocess.run([exe], check=True, capture_output=True, text=True).stdout


def _sizes_in_tiles(P, tiles):
    """Six tensors, mostly one of them, that the planner cuts into this many tiles."""
    import paper_2302_12445_amd as dear
    for big in range((tiles - P - 16) * 4096 + 77, (tiles + 2) * 4096, 1024):
        sizes = [7, 9_000, 33, big, 3, 4095]
        if len(dear.dear_plan_tiles(dear.dear_plan(sizes, P, dear.DEAR_NO_LIMIT, 4))[0]) == tiles:
            return sizes
    raise AssertionError("no plan of %d tiles for %d workers" % (tiles, P))


# one below each line of the rule and on it: by workers, the limit of few workers, and two workers, who never go in eighths
@pytest.mark.gpu
@pytest.mark.parametrize("P,tiles", [(2, 2048), (3, 2047), (3, 2048), (4, 4999), (4, 5000), (5, 2047), (5, 5000), (8, 2050), (11, 2047), (12, 1599),
                                     (12, 1600), (23, 1599), (24, 959), (24, 960), (33, 1025), (64, 959), (64, 963)])
def test_around_the_lines_of_the_rule(P, tiles):
    from test_gpu_parity import Pair, say, small_workload
    import workloads as W
    say("case: all-gather in eighths, P=%d, %d tiles" % (P, tiles))
    pair = Pair(small_workload(_sizes_in_tiles(P, tiles), P, W.NO_LIMIT, "f32" if P % 2 else "bf16"))
    for route in ("calls", "iteration"):
        pair.run(iterations=1, route=route, fused=route == "iteration")
    pair.close()


# replicas on lines; alike, off the lines; each elsewhere (parts as they fall), as they do for two workers
@pytest.mark.gpu
@pytest.mark.parametrize("starts", [(0, 0, 0, 0), (4, 4, 4, 4), (28, 28, 28, 28), (0, 12, 20, 4)])
@pytest.mark.parametrize("workers", [(0, 4), (1, 3), (1, 2)])
def test_replicas_alike_and_not(starts, workers):
    import numpy as np
    import oracle
    import torch
    import paper_2302_12445_amd as dear
    import workloads as W
    from test_gpu_parity import DEV, _bits, say
    say("case: all-gather in eighths, tensors at %s of a line, workers %s" % (starts, workers))
    sizes, P = [9_000_003, 70_001], 4
    op, plan = oracle.plan(sizes, P, W.NO_LIMIT, 4), dear.dear_plan(sizes, P, W.NO_LIMIT, 4)
    assert 2048 <= len(dear.dear_plan_tiles(plan)[0]) < 5000
    bufs = [[torch.full((n + 64,), 7.0, device=DEV) for n in sizes] for _ in range(P)]
    ptrs = [b.data_ptr() + 4 * starts[p] for p in range(P) for b in bufs[p]]
    ctx = dear.dear_ctx_create(plan, dear.DEAR_F32, ptrs, ptrs)
    shards = torch.randn(P, op.total_shard_len, generator=torch.Generator().manual_seed(5))
    dev = shards.to(DEV)
    dear.dear_all_gather_workers(ctx, -1, dev.data_ptr(), workers[0], workers[1])
    torch.cuda.synchronize()
    params = [[np.full(n, 7.0, np.float32) for n in sizes] for _ in range(P)]
    oracle.all_gather(op, -1, shards.numpy(), params, workers=range(workers[0], workers[0] + workers[1]))
    for p in range(P):
        for got, want in zip(bufs[p], params[p]):
            whole = np.full(got.numel(), 7.0, np.float32)
            whole[starts[p]:starts[p] + want.size] = want
            assert np.array_equal(_bits(got.cpu().numpy()), _bits(whole)), p
    ctx.destroy()
