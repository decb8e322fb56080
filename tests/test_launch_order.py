"""Which workgroup takes what: the rules on the host, and launches at the sizes where the all-gather's numbering, the form of
the bf16 reduce-scatter and the number of an iteration's launches change, against the oracle."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

W_NO_LIMIT = (1 << 63) - 1
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_order_and_rules_on_the_host(tmp_path):
    exe = str(tmp_path / "launch_order")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2302_12445_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "launch_order.cpp"), "-o", exe], check=True)
    assert "launch_order: ok" in subprocess.run([exe], check=True, capture_output=True, text=True).stdout


def test_pointer_arrays_are_what_ctypes_makes_of_the_addresses():
    import ctypes as C
    import numpy as np
    from paper_2302_12445_amd import binding as B
    far = (1 << 64) - 256
    for a in ([], [0], [far, 16], (1 << 40, 32), [None, 48], [-16], [True], np.array([64, 1 << 45], np.int64), np.array([far], np.uint64), b"ab"):
        assert list(B._pointers(a)) == list((C.c_void_p * len(a))(*[int(x) if isinstance(x, np.integer) else x for x in a]))
    for a in (["x"], [1.5]):
        with pytest.raises(TypeError):
            B._pointers(a)


def test_stream_handle_without_torchs_private_name(monkeypatch):
    import torch
    from types import SimpleNamespace
    from paper_2302_12445_amd import emulation
    monkeypatch.setattr(emulation, "_raw_current_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=4711))
    assert emulation._stream_handle(None) == 4711
    assert emulation._stream_handle(SimpleNamespace(cuda_stream=5)) == 5


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


# one launch / several: below and above the limit for the replica count, few-replica calls with one and two workgroups per
# CU, few tiles for many replicas, thousands of open tiles, run ends of every alignment
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P,sizes", [
    ("f32", 1, [1]), ("f32", 1, [4_100_003, 5]), ("f32", 2, [4_000_000, 300_001]), ("f32", 3, [25_000_001, 77]), ("f32", 5, [1_790_000]),
    ("f32", 5, [1_810_001]), ("f32", 8, [740_000]), ("f32", 8, [760_000]), ("f32", 8, [970_000]), ("f32", 8, [1_030_000]), ("f32", 11, [530_003]), ("f32", 16, [701] * 900), ("f32", 33, [77, 200] * 40), ("f32", 33, [77, 200] * 10),
    ("f32", 12, [33, 5, 4100]), ("f32", 26, [2000] * 150),
    ("bf16", 1, [9, 4096, 3]), ("bf16", 2, [1_650_000, 9]), ("bf16", 2, [25_000_100]), ("bf16", 7, [1_600_003, 33]), ("bf16", 8, [1_500_000 + 4096]),
    ("bf16", 5, [507 * 4096]), ("bf16", 5, [509 * 4096]), ("bf16", 8, [2600] * 400), ("bf16", 33, [2000] * 150), ("bf16", 9, [50_000, 3]),
    ("bf16", 12, [577_777, 3]), ("bf16", 24, [1000, 64, 33] * 300), ("bf16", 6, list(range(1, 19)) + [4096 + k for k in range(9)] + [2047, 2049]),
])
def test_iteration_in_one_launch(dtype, P, sizes):
    from test_gpu_parity import Pair, say, small_workload
    import workloads as W
    say("case: iteration, %s, P=%d, %d tensors, %d elements" % (dtype, P, len(sizes), sum(sizes)))
    pair = Pair(small_workload(sizes, P, W.NO_LIMIT, dtype))
    pair.run(iterations=2 if sum(sizes) * P < 20_000_000 else 1, route="iteration")
    pair.run(iterations=1, route="iteration", fused=True)
    pair.run(iterations=1, route="iteration", width=64)
    pair.close()


# one bucket beyond 8192 tiles: pieces that begin inside a layer and a shard
@pytest.mark.gpu
@pytest.mark.parametrize("dtype,P,thr,width", [("f32", 5, None, 0), ("bf16", 3, None, 0), ("bf16", 5, 40_000_000, 0), ("bf16", 3, None, 300)])
def test_iteration_over_a_bucket_in_pieces(dtype, P, thr, width):
    from test_gpu_parity import Pair, say, small_workload
    import workloads as W
    say("case: one bucket in pieces, %s, P=%d, width %d" % (dtype, P, width))
    pair = Pair(small_workload([17_000_001, 3, 20_100_077], P, thr or W.NO_LIMIT, dtype))
    pair.run(iterations=1, route="iteration", width=width)
    pair.run(iterations=1, route="iteration", fused=True, width=width)
    pair.close()


# pieces that begin inside a run whose all-gather's cuts are moved to the replicas' 128-byte lines: every cut is where the one
# all-gather over the whole bucket has it, and nothing around the tensors is written
@pytest.mark.gpu
@pytest.mark.parametrize("starts,width", [((4, 4, 4), 0), ((28, 28, 28), 0), ((0, 12, 20), 0), ((16, 4, 28), 300)])
def test_pieces_of_runs_with_moved_cuts(starts, width):
    import torch
    import paper_2302_12445_amd as dear
    from paper_2302_12445_amd import binding as B
    print("case: pieces, tensors at %s of a line, width %d" % (starts, width), flush=True)
    sizes, P = [17_000_001, 20_100_077], 3
    plan = dear.dear_plan(sizes, P, W_NO_LIMIT, 2)
    gen = torch.Generator("cuda:0").manual_seed(sum(starts))
    grads = [[torch.randn(n, device="cuda:0", generator=gen).to(torch.bfloat16) for n in sizes] for _ in range(P)]
    w0 = torch.randn(P, plan.total_shard_len, device="cuda:0", generator=gen)
    got = []
    for whole in (False, True):
        params = [[torch.full((n + 96,), 7.0, device="cuda:0") for n in sizes] for _ in range(P)]
        ctx = dear.dear_ctx_create(plan, B.DEAR_BF16, [t.data_ptr() for rep in grads for t in rep],
                                   [t.data_ptr() + 4 * (32 + starts[p]) for p, rep in enumerate(params) for t in rep])
        g, w, v = torch.zeros_like(w0), w0.clone(), w0 * 0.25
        if whole:  # a launch of each, over all tiles
            dear.dear_reduce_scatter(ctx, -1, g.data_ptr())
            dear.dear_shard_update(ctx, -1, g.data_ptr(), w.data_ptr(), v.data_ptr(), 0.1, 0.9)
            dear.dear_all_gather(ctx, -1, w.data_ptr())
        else:
            dear.dear_ctx_set_max_workgroups(ctx, width)
            dear.dear_iteration(ctx, -1, g.data_ptr(), w.data_ptr(), v.data_ptr(), 0.1, 0.9)
        torch.cuda.synchronize()
        got.append([g, w, v] + [t for rep in params for t in rep])
        ctx.destroy()
    for a, b in zip(*got):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))
    for p, t in enumerate(got[0][3::2]):
        assert bool((t[:32 + starts[p]] == 7.0).all()) and bool((t[32 + starts[p] + sizes[0]:] == 7.0).all())
        assert int((t[32 + starts[p]:32 + starts[p] + sizes[0]] == 7.0).sum()) < 10


# tables of one upload piece, of several and of more than go in pieces, nothing waited for between calls; tiles cut on the host
# (tensors of about a tile) and on the device (long ones)
@pytest.mark.gpu
def test_static_calls_back_to_back():
    import torch
    import paper_2302_12445_amd as dear
    from paper_2302_12445_amd import binding as B
    from paper_2302_12445_amd.emulation import EmulatedWorkers
    ems = [EmulatedWorkers([n + 7 * l for l in range(L)], P, dtype, thr, "cuda:0")
           for n, L, P, dtype, thr in ((1000, 5, 4, "f32", 9000), (90_000, 3, 2, "bf16", W_NO_LIMIT), (1000, 300, 8, "bf16", 40_000), (1000, 1, 3, "f32", 0),
                                       (20_000, 130, 4, "f32", 900_000), (1000, 500, 9, "f32", W_NO_LIMIT), (1000, 700, 16, "f32", 60_000))]
    side = torch.cuda.Stream()
    outs = []
    for em in ems:
        for rep in em.grads:
            rep[0]._base.normal_(generator=torch.Generator("cuda:0").manual_seed(len(outs)))
        em.reduce_scatter()
        outs.append(torch.full_like(em.shard_grad, 7.0))
    side.wait_stream(torch.cuda.current_stream())
    for em, out in zip(ems, outs):
        print("case: static reduce-scatter, %d layers, P=%d" % (len(em.sizes), em.P), flush=True)
        dear.dear_reduce_scatter_static(em.plan, B.DEAR_F32 if em.grad_dtype == "f32" else B.DEAR_BF16,
                                        [t.data_ptr() for rep in em.grads for t in rep], -1, out.data_ptr(), side.cuda_stream)
    side.synchronize()
    for em, out in zip(ems, outs):
        assert torch.equal(out.view(torch.int32), em.shard_grad.view(torch.int32))


@pytest.mark.gpu
def test_static_call_refuses_a_captured_stream():
    import torch
    import paper_2302_12445_amd as dear
    from paper_2302_12445_amd import binding as B
    from paper_2302_12445_amd.emulation import EmulatedWorkers
    em = EmulatedWorkers([5000, 77], 3, "f32", W_NO_LIMIT, "cuda:0")
    ptrs = [t.data_ptr() for rep in em.grads for t in rep]
    side, x = torch.cuda.Stream(), torch.zeros(4, device="cuda:0")
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        x.add_(1)
        with pytest.raises(dear.DearError) as e:
            dear.dear_reduce_scatter_static(em.plan, B.DEAR_F32, ptrs, -1, em.shard_grad.data_ptr(), side.cuda_stream)
        assert e.value.status == B.DEAR_EHIP
    for n in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert x.tolist() == [n] * 4
    dear.dear_reduce_scatter_static(em.plan, B.DEAR_F32, ptrs, -1, em.shard_grad.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()


# quarters of tiles: runs that begin and end at every element of a vector, at a part's ends, within old shards of other lengths
@pytest.mark.gpu
@pytest.mark.parametrize("P,thr_from,thr_to", [(1, W_NO_LIMIT, 0), (3, 0, 30_000), (7, 9000, W_NO_LIMIT), (5, W_NO_LIMIT, 60_001)])
def test_copies_between_layouts(P, thr_from, thr_to):
    import torch
    import paper_2302_12445_amd as dear
    from paper_2302_12445_amd.emulation import EmulatedWorkers
    print("case: copies between layouts, P=%d" % P, flush=True)
    sizes = list(range(1, 12)) + [1024 * k + j for k in (1, 2, 3, 4) for j in (-1, 0, 1, 2, 3)] + [30_001, 5, 12_289]
    gen = torch.Generator("cuda:0").manual_seed(P)
    old = EmulatedWorkers(sizes, P, "f32", thr_from, "cuda:0")
    new = EmulatedWorkers(sizes, P, "f32", thr_to, "cuda:0")
    for em in (old, new):
        em.params[P - 1][0]._base.normal_(generator=gen.manual_seed(P))
        em.shard_param.fill_(float("nan"))
        em.scatter_params(P - 1)
        for layer, t in enumerate(em.params[P - 1]):      # slot of every element, by the plan's own numbers
            b = em.plan.layer_bucket[layer]
            S, base = em.plan.bucket_shard_len[b], em.plan.bucket_shard_base[b]
            e = em.plan.layer_offset[layer] + torch.arange(t.numel(), device="cuda:0")
            assert torch.equal(em.shard_param[e // S, base + e % S], t)
        assert int(em.shard_param.isnan().sum()) == 0 and float(em.shard_param.double().abs().sum()) > 0
        assert int((em.shard_param != 0).sum()) <= sum(sizes)     # padding slots are +0
    out = torch.full_like(new.shard_param, float("nan"))
    dear.dear_reshard(old.ctx, new.ctx, old.shard_param.data_ptr(), out.data_ptr())
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int32), new.shard_param.view(torch.int32))


# update and all-gather in one call, on both sides of the limits: quarters of tiles and whole ones, full and open ones, one kernel
# and two (the limits themselves are pinned in native/launch_rules.cpp)
@pytest.mark.gpu
@pytest.mark.parametrize("P,sizes", [(1, [5]), (2, [141 * 4096, 77]), (2, [146 * 4096 + 1]), (3, [110 * 4096 - 5]), (7, [171 * 4096, 9]), (16, [9001] * 40),
                                     (3, [300, 701, 64] * 150), (4, [2100] * 60), (4, [2100] * 400), (8, [30, 5000, 7] * 150), (26, [450_000]), (26, [333] * 90),
                                     (5, [2_000_003]), (5, [4_010_001, 33]), (8, [900] * 700), (12, [1_700_000])])
def test_update_all_gather_forms(P, sizes):
    from test_gpu_parity import Pair, say, small_workload
    import workloads as W
    say("case: update + all-gather, P=%d, %d tensors, %d elements" % (P, len(sizes), sum(sizes)))
    pair = Pair(small_workload(sizes, P, W.NO_LIMIT))
    pair.run(iterations=1, fused_gather=True)
    pair.run(iterations=1, fused_gather=True, width=50)
    pair.close()
