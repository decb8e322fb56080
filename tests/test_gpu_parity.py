"""GPU parity: the HIP path through the C ABI against the CPU oracle, element by element
on the same seeded inputs.  fp32 gradients: bit-exact.  bf16 gradients: the shard values
are fp32 on both sides and the ring order is fixed, so bits are compared too (the stated
acceptance floor of 2 bf16 ULP is asserted separately as the weaker bound).  Bucket and
shard indexing: bit-exact through the positions of the values."""
from __future__ import annotations

import ctypes as C
import sys

import numpy as np
import pytest
import torch

import oracle
import workloads as W
from helpers import bf16_ulp, separate_calls, small_workload, split_np, to_numpy

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _bits(a: np.ndarray) -> np.ndarray:
    return np.ascontiguousarray(a).view(np.uint32)


class Pair:
    """The same problem on both sides: EmulatedWorkers on the GPU, numpy + oracle on the CPU."""

    def __init__(self, w: W.Workload, layout="flat", plan=None, oracle_plan=None):
        """plan / oracle_plan: the two sides' own plans when the grouping is not the
        workload's threshold rule (each side builds its plan with its own planner)."""
        from paper_2302_12445_amd.emulation import EmulatedWorkers
        self.w = w
        self.em = EmulatedWorkers(w.sizes, w.P, w.grad_dtype, w.threshold_bytes, DEV, layout, plan)
        self.op = oracle_plan if oracle_plan is not None else oracle.plan(
            w.sizes, w.P, w.threshold_bytes, w.grad_elem_bytes)
        row = self.op.total_shard_len
        assert row == self.em.plan.total_shard_len
        self.sg = np.zeros((w.P, row), np.float32)
        self.sp = np.zeros_like(self.sg)
        self.sm = np.zeros_like(self.sg)
        flat = W.make_flat_param(w)
        self.params = [split_np(to_numpy(flat).copy(), w.sizes) for _ in range(w.P)]
        for p in range(w.P):
            self.em.load_dense(self.em.params[p], flat.to(DEV))
        self.grads = None

    def seed_shards(self):
        oracle.scatter_params(self.op, self.params, 0, self.sp)
        self.em.shard_param.fill_(float("nan"))
        self.em.scatter_params(0)
        self.compare_buffer("scatter_params", self.em.shard_param, self.sp)

    def load_grads(self, it, flats=None):
        w = self.w
        if flats is None:
            flats = [W.make_flat_grad(w, p, it) for p in range(w.P)]
        self.grads = [split_np(to_numpy(f), w.sizes) for f in flats]
        for p in range(w.P):
            self.em.load_dense(self.em.grads[p], flats[p].to(DEV))

    def compare_buffer(self, what, dev: torch.Tensor, host: np.ndarray):
        got = dev.cpu().numpy()
        same = _bits(got) == _bits(host)
        if not same.all():
            idx = np.argwhere(~same)[:5]
            raise AssertionError("%s: %d of %d slots differ, first at %s: got %s want %s" % (
                what, (~same).sum(), same.size, idx.tolist(),
                [got[tuple(i)] for i in idx], [host[tuple(i)] for i in idx]))

    def compare_params(self, what):
        for p in range(self.w.P):
            for l in range(self.w.n_layers):
                got = self.em.params[p][l].cpu().numpy()
                want = self.params[p][l]
                if not np.array_equal(_bits(got), _bits(want)):
                    bad = np.argwhere(_bits(got) != _bits(want))[:5].ravel()
                    raise AssertionError("%s: worker %d layer %d differs at %s: got %s want %s" % (
                        what, p, l, bad.tolist(), got[bad], want[bad]))

    def oracle_iteration(self):
        w = self.w
        oracle.reduce_scatter(self.op, -1, self.grads, self.sg)
        oracle.shard_update(self.op, -1, self.sg, self.sp, self.sm, w.lr, w.momentum)
        oracle.all_gather(self.op, -1, self.sp, self.params)

    def run(self, iterations=3, per_bucket=True, poison=True, stream=None, fused=False, width=0, priority=0,
            fused_gather=False, route="calls"):
        """route "calls": the library's separate calls, as per_bucket, fused and fused_gather say;
        "iteration": EmulatedWorkers.iteration, one library call that chooses its own launches."""
        assert route in ("calls", "iteration")
        w, em = self.w, self.em
        em.set_max_workgroups(width)
        em.set_wave_priority(priority)
        self.seed_shards()
        for it in range(iterations):
            self.load_grads(it)
            if poison:  # nothing may survive from before: every slot and element is rewritten
                em.shard_grad.fill_(float("nan"))
                for p in range(w.P):
                    for t in em.params[p]:
                        t.fill_(float("nan"))
            torch.cuda.synchronize()
            if route == "calls":
                separate_calls(em, w.lr, w.momentum, per_bucket, fused, fused_gather, stream)
            else:
                em.iteration(w.lr, w.momentum, per_bucket=per_bucket, stream=stream, fused_update=fused,
                             fused_gather=fused_gather)
            torch.cuda.synchronize()
            self.oracle_iteration()
            if not fused:  # the fused kernel never writes the averaged gradient
                self.compare_buffer("shard_grad it%d" % it, em.shard_grad, self.sg)
            self.compare_buffer("shard_mom it%d" % it, em.shard_mom, self.sm)
            self.compare_buffer("shard_param it%d" % it, em.shard_param, self.sp)
            self.compare_params("params it%d" % it)

    def close(self):
        self.em.close()


RAGGED = [4097, 3, 8191, 4096, 1, 12289, 7, 30001, 64, 513]


@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_tiny_config_three_iterations(route):
    say("case: tiny config, per-bucket launches")
    pr = Pair(W.get_workload("tiny"))
    assert pr.em.plan.n_buckets == 5
    pr.run(3, per_bucket=True, route=route)
    pr.close()


def test_tiny_config_all_buckets_in_one_launch():
    say("case: tiny config, bucket=-1 launches, separate allocations")
    pr = Pair(W.get_workload("tiny"), layout="separate")
    pr.run(3, per_bucket=False)
    pr.close()


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 8, 9, 12, 16, 24, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_ragged_layers_all_worker_counts(P, dtype, route):
    say("case: ragged layers P=%d %s" % (P, dtype))
    g = 4 if dtype == "f32" else 2
    w = small_workload(RAGGED, P, 21000 * g, dtype, index=10 + P)
    pr = Pair(w)
    assert pr.em.plan.n_buckets >= 3
    pr.run(2 if P > 16 else 3, per_bucket=(P % 2 == 0), route=route)
    pr.close()


@pytest.mark.parametrize("P", [1, 2, 3, 4, 8, 9, 12, 64])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_fused_reduce_scatter_update(P, dtype, route):
    """dear_reduce_scatter_update, and dear_iteration without a gradient buffer, must leave the same bits in the
    parameter and momentum shards as dear_reduce_scatter followed by dear_shard_update (both compared with the oracle)."""
    say("case: fused RS+update P=%d %s" % (P, dtype))
    g = 4 if dtype == "f32" else 2
    w = small_workload(RAGGED + [70001, 2], P, 36000 * g, dtype, index=110 + P)
    pr = Pair(w)
    pr.run(3, per_bucket=(P % 2 == 1), fused=True, route=route)
    pr.close()


@pytest.mark.parametrize("width", [1, 3, 64, 256])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_bounded_grid_gives_the_same_bits(width, dtype, route):
    """A bounded grid (workgroups striding over the work items) is only a launch shape."""
    say("case: bounded grid width=%d %s" % (width, dtype))
    g = 4 if dtype == "f32" else 2
    w = small_workload(RAGGED + [300_001], 4, 40000 * g, dtype, index=120 + width)
    pr = Pair(w)
    pr.run(2, per_bucket=(width != 3), fused=(width == 64), width=width, priority=width % 4, route=route)
    pr.close()


@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_fused_tiny_and_many_tiles(route):
    say("case: fused RS+update, tiny config and many tiles")
    pr = Pair(W.get_workload("tiny"))
    pr.run(3, fused=True, route=route)
    pr.close()
    w = small_workload([1_000_003, 5, 65_537, 250_001, 2], 8, 1_100_000 * 2, "bf16", index=42, std=1e-3)
    pr = Pair(w)
    pr.run(2, fused=True, route=route)
    pr.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_single_bucket_and_no_fusion(dtype, route):
    g = 4 if dtype == "f32" else 2
    for thr in (W.NO_LIMIT, 0):
        say("case: threshold %d %s" % (thr, dtype))
        w = small_workload(RAGGED, 4, thr, dtype, index=31)
        pr = Pair(w)
        assert pr.em.plan.n_buckets == (1 if thr else len(RAGGED))
        pr.run(2, route=route)
        pr.close()
    del g


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_many_tiles_per_shard(dtype, route):
    """Several hundred tiles per shard, layer starts that are odd in the bucket, a layer
    spanning several shards."""
    say("case: many tiles %s" % dtype)
    g = 4 if dtype == "f32" else 2
    w = small_workload([1_000_003, 5, 65_537, 250_001, 2], 8, 1_100_000 * g, dtype, index=41, std=1e-3)
    pr = Pair(w)
    pr.run(2, route=route)
    pr.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("layers_per_bucket", [4, 3])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_fixed_layers_plan(dtype, layers_per_bucket, route):
    """The fixed-number-of-layers grouping of the tensor-fusion study (Section VI-G) drives the
    same kernels: the library's plan and the oracle's own fixed-layers plan, bit for bit over
    the shards of every worker and the parameters of every replica, three iterations."""
    import paper_2302_12445_amd as dear
    say("case: fixed-layers plan, %d layers per bucket, %s" % (layers_per_bucket, dtype))
    g = 4 if dtype == "f32" else 2
    w = small_workload(RAGGED, 4, W.NO_LIMIT, dtype, index=51)
    plan = dear.dear_plan_fixed_layers(w.sizes, w.P, layers_per_bucket, g)
    op = oracle.plan_fixed_layers(w.sizes, w.P, layers_per_bucket, g)
    assert plan.n_buckets == op.n_buckets == -(-len(RAGGED) // layers_per_bucket)
    pr = Pair(w, plan=plan, oracle_plan=op)
    pr.run(3, route=route)
    pr.run(1, fused=True, route=route)
    pr.close()


def test_fixed_layers_plan_resnet50_shape():
    """Four layers per bucket (the paper's number) on the ResNet-50 tensor list: 41 buckets of
    very uneven size, one launch per bucket."""
    import paper_2302_12445_amd as dear
    say("case: fixed-layers plan, resnet50 shape")
    w = W.get_workload("resnet50")
    plan = dear.dear_plan_fixed_layers(w.sizes, w.P, 4, 4)
    op = oracle.plan_fixed_layers(w.sizes, w.P, 4, 4)
    assert plan.n_buckets == op.n_buckets == 41
    pr = Pair(w, plan=plan, oracle_plan=op)
    pr.run(1)
    pr.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P,width", [(1, 0), (4, 0), (8, 5), (13, 0)])
def test_fused_update_all_gather_gives_the_same_bits(P, width, dtype):
    """dear_update_all_gather: update and all-gather of a bucket in one kernel; shard buffers
    (padding slots included) and every replica's parameters as from the two separate calls."""
    say("case: fused update+all-gather P=%d width=%d %s" % (P, width, dtype))
    g = 4 if dtype == "f32" else 2
    w = small_workload(RAGGED + [100_003], P, 30000 * g, dtype, index=140 + P)
    pr = Pair(w)
    pr.run(3, fused_gather=True, width=width, priority=P % 4)
    pr.run(1, per_bucket=False, fused_gather=True)
    pr.close()


def test_signed_zero_nan_inf():
    say("case: signed zeros, NaN, Inf")
    w = small_workload([37, 4100], 4, W.NO_LIMIT, "f32", index=61)
    pr = Pair(w)
    pr.seed_shards()
    flats = [torch.full((w.N,), -0.0) for _ in range(4)]
    pr.load_grads(0, flats)
    pr.em.shard_grad.fill_(float("nan"))
    pr.em.reduce_scatter(-1)
    oracle.reduce_scatter(pr.op, -1, pr.grads, pr.sg)
    pr.compare_buffer("negative zeros", pr.em.shard_grad, pr.sg)
    assert (_bits(pr.sg[0, :37]) == 0x80000000).all()
    flats = [W.make_flat_grad(w, p, 0) for p in range(4)]
    flats[1][5] = float("inf")
    flats[2][6] = float("-inf")
    flats[3][7] = float("nan")
    flats[0][4000] = float("inf")
    flats[1][4000] = float("-inf")
    pr.load_grads(0, flats)
    pr.em.reduce_scatter(-1)
    oracle.reduce_scatter(pr.op, -1, pr.grads, pr.sg)
    got = pr.em.shard_grad.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(pr.sg))
    ok = ~np.isnan(got)
    assert np.array_equal(_bits(got[ok]), _bits(pr.sg[ok]))
    pr.close()


def test_denormals_are_kept():
    say("case: denormal gradients")
    w = small_workload([4096 + 9], 2, W.NO_LIMIT, "f32", index=62)
    pr = Pair(w)
    pr.seed_shards()
    tiny = np.float32(1e-41)
    flats = [torch.full((w.N,), float(tiny)), torch.full((w.N,), float(tiny) * 3)]
    pr.load_grads(0, flats)
    pr.em.reduce_scatter(-1)
    oracle.reduce_scatter(pr.op, -1, pr.grads, pr.sg)
    assert pr.sg[0, 0] != 0.0
    pr.compare_buffer("denormals", pr.em.shard_grad, pr.sg)
    pr.close()


def test_bf16_within_two_ulp_of_exact_mean():
    """The acceptance floor stated for bf16 gradients, checked against the exact mean."""
    say("case: bf16 two-ULP floor")
    w = small_workload([5000, 123], 8, W.NO_LIMIT, "bf16", index=63, std=1e-3)
    pr = Pair(w)
    pr.seed_shards()
    flats = [W.make_flat_grad(w, p, 0) for p in range(8)]
    pr.load_grads(0, flats)
    pr.em.reduce_scatter(-1)
    pr.em.shard_param.copy_(pr.em.shard_grad)
    pr.em.all_gather(-1)
    torch.cuda.synchronize()
    mean = torch.stack([f.double() for f in flats]).sum(0).numpy() / 8
    got = pr.em.dense(pr.em.params[3]).cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - mean) <= 2 * bf16_ulp(mean))
    pr.close()


def test_side_stream_and_argument_errors():
    import paper_2302_12445_amd as dear
    from paper_2302_12445_amd import binding
    say("case: side stream, error codes")
    w = small_workload(RAGGED, 4, 21000 * 4, "f32", index=71)
    pr = Pair(w)
    side = torch.cuda.Stream()
    pr.run(2, stream=side)
    pr.run(1, stream=side, route="iteration")
    em = pr.em
    lib = dear.load_library()
    h = em.ctx.handle
    sg, sp, sm = em.shard_grad.data_ptr(), em.shard_param.data_ptr(), em.shard_mom.data_ptr()
    nb = em.plan.n_buckets
    assert lib.dear_reduce_scatter(h, nb, C.c_void_p(sg), None) == binding.DEAR_ERANGE
    assert lib.dear_reduce_scatter(h, -2, C.c_void_p(sg), None) == binding.DEAR_ERANGE
    assert lib.dear_reduce_scatter(h, 0, C.c_void_p(sg + 64), None) == binding.DEAR_EALIGN
    assert lib.dear_reduce_scatter(h, 0, None, None) == binding.DEAR_EINVAL
    assert lib.dear_all_gather(h, nb, C.c_void_p(sp), None) == binding.DEAR_ERANGE
    assert lib.dear_all_gather(h, 0, C.c_void_p(sp + 4), None) == binding.DEAR_EALIGN
    assert lib.dear_shard_update(h, 0, C.c_void_p(sg), C.c_void_p(sg), C.c_void_p(sm), 0.1, 0.9, None) == binding.DEAR_EINVAL
    assert lib.dear_shard_update(h, nb, C.c_void_p(sg), C.c_void_p(sp), C.c_void_p(sm), 0.1, 0.9, None) == binding.DEAR_ERANGE
    assert lib.dear_scatter_params(h, 4, C.c_void_p(sp), None) == binding.DEAR_ERANGE
    assert lib.dear_scatter_params(h, -1, C.c_void_p(sp), None) == binding.DEAR_ERANGE
    torch.cuda.synchronize()
    # nothing was launched by the failing calls: state still equals the oracle's
    pr.compare_buffer("after errors", em.shard_param, pr.sp)
    pr.close()


@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_resnet50_config_one_iteration(route):
    """Config 2 at full size: 161 tensors, 5 buckets of up to 76 small tensors, P = 8."""
    say("case: resnet50 full size")
    pr = Pair(W.get_workload("resnet50"))
    assert pr.em.plan.n_buckets == 5
    pr.run(1, route=route)
    pr.close()


@pytest.mark.parametrize("name", ["densenet201", "inception_v4"])
@pytest.mark.parametrize("route", ["calls", "iteration"])
def test_many_small_tensors_full_size(name, route):
    """The paper's other two CNNs at full size: 604 / 449 tensors, hundreds of them a few
    hundred elements long, so most tiles are short runs and edge vectors."""
    say("case: %s full size" % name)
    pr = Pair(W.get_workload(name))
    pr.run(1, fused=(name == "inception_v4"), route=route)
    pr.close()


def test_random_configurations():
    """Seeded random layer lists, worker counts, thresholds, gradient types, launch widths,
    fused or not, flat or separate allocations: each compared bit for bit with the oracle."""
    rng = np.random.default_rng(20230212)
    picks = [1, 2, 3, 5, 7, 8, 31, 32, 33, 63, 64, 65, 100, 255, 256, 257, 1000, 1023, 1024, 1025,
             4095, 4096, 4097, 8191, 8192, 8193, 12289, 20000, 40001]
    for case in range(40):
        L = int(rng.integers(1, 14))
        sizes = [int(rng.choice(picks)) for _ in range(L)]
        if rng.random() < 0.3:
            sizes[int(rng.integers(0, L))] = int(rng.integers(50000, 300000))
        P = int(rng.choice([1, 2, 3, 4, 5, 6, 7, 8, 9, 12, 16, 17, 24, 33]))
        dtype = str(rng.choice(["f32", "bf16"]))
        g = 4 if dtype == "f32" else 2
        thr = int(rng.choice([0, 64 * g, 5000 * g, 30000 * g, 200000 * g, W.NO_LIMIT]))
        width = int(rng.choice([0, 0, 1, 2, 7, 64, 256]))
        fused = bool(rng.random() < 0.5)
        per_bucket = bool(rng.random() < 0.5)
        layout = str(rng.choice(["flat", "separate"]))
        route = ["calls", "iteration"][case % 2]
        say("case: random %d sizes=%s P=%d %s thr=%d width=%d fused=%d per_bucket=%d %s %s" % (
            case, sizes, P, dtype, thr, width, fused, per_bucket, layout, route))
        pr = Pair(small_workload(sizes, P, thr, dtype, index=1000 + case), layout=layout)
        pr.run(2, per_bucket=per_bucket, fused=fused, width=width, priority=case // 2 % 4, route=route)
        pr.close()


@pytest.mark.parametrize("n", [1 << 22, (1 << 22) + 1, (1 << 22) - 4096, 2 * (1 << 22) + 70001, 5])
def test_all_gather_whole_and_short_chunks(n):
    """The all-gather orders its work in chunks of 4 Mi elements with a short last one: around the
    chunk's edges, for all replicas and for a range of them; the others stay as they are."""
    say("case: all-gather, %d elements in one layer and a ragged one" % n)
    pair = Pair(small_workload([n, 777], 3, W.NO_LIMIT))
    pair.seed_shards()
    em = pair.em
    for first, count in ((0, 3), (1, 2), (2, 1)):
        em.shard_param.copy_(torch.randn(em.shard_param.shape, generator=torch.Generator().manual_seed(n + first)))
        for rep in em.params:
            for t in rep:
                t.fill_(7.0)
        for rep in pair.params:
            for t in rep:
                t.fill(7.0)
        torch.cuda.synchronize()
        from paper_2302_12445_amd import dear_all_gather_workers
        dear_all_gather_workers(em.ctx, -1, em.shard_param.data_ptr(), first, count)
        torch.cuda.synchronize()
        oracle.all_gather(pair.op, -1, to_numpy(em.shard_param), pair.params, workers=range(first, first + count))
        pair.compare_params("workers %d..%d" % (first, first + count - 1))
    pair.close()


@pytest.mark.parametrize("dtype,keep,width", [("f32", True, 0), ("f32", False, 0), ("bf16", True, 0),
                                              ("bf16", False, 5), ("f32", True, 7)])
def test_iteration_call_of_one_bucket_and_of_several_groups(dtype, keep, width):
    """dear_iteration on one bucket touches nothing else, and on a plan whose buckets do not all fit
    one pair of launches (8192 tiles of 4096 elements) equals the three calls."""
    from paper_2302_12445_amd import dear_iteration
    say("case: iteration call, %s, keep %s, width %d" % (dtype, keep, width))
    for sizes, P, bucket in ((RAGGED, 5, 3), ([12_000_003, 12_000_001, 12_000_000, 70], 2, -1)):
        pair = Pair(small_workload(sizes, P, 0, dtype))
        em, op, w = pair.em, pair.op, pair.w
        em.set_max_workgroups(width)
        pair.seed_shards()
        pair.load_grads(0)
        pair.sg[...] = -3.0
        em.shard_grad.fill_(-3.0)
        dear_iteration(em.ctx, bucket, em.shard_grad.data_ptr() if keep else None, em.shard_param.data_ptr(),
                       em.shard_mom.data_ptr(), w.lr, w.momentum)
        torch.cuda.synchronize()
        kept = pair.sg.copy()
        oracle.reduce_scatter(op, bucket, pair.grads, pair.sg)
        oracle.shard_update(op, bucket, pair.sg, pair.sp, pair.sm, w.lr, w.momentum)
        oracle.all_gather(op, bucket, pair.sp, pair.params)
        pair.compare_buffer("shard_grad", em.shard_grad, pair.sg if keep else kept)
        pair.compare_buffer("shard_mom", em.shard_mom, pair.sm)
        pair.compare_buffer("shard_param", em.shard_param, pair.sp)
        pair.compare_params("params")
        pair.close()


@pytest.mark.parametrize("dtype,P,n", [("f32", 25, 2048 * 4096), ("f32", 24, 2000 * 4096), ("bf16", 48, 2048 * 4096)])
def test_iteration_call_with_many_replicas(dtype, P, n):
    """From 96 gradient bytes per element and 2048 tiles on dear_iteration updates in a launch of its own if the
    averaged gradients are wanted; below, and without them, inside the reduce-scatter."""
    say("case: iteration call, P=%d, %d elements, %s" % (P, n, dtype))
    pair = Pair(small_workload([n - 33, 33], P, W.NO_LIMIT, dtype))
    pair.run(iterations=1, route="iteration")
    pair.run(iterations=1, route="iteration", width=300)
    pair.close()


@pytest.mark.parametrize("P,n", [(4, 1100 * 4096), (5, 831 * 4096), (5, 830 * 4096), (8, 519 * 4096), (8, 518 * 4096), (16, 260 * 4096),
                                 (16, 259 * 4096), (24, 225 * 4096), (24, 224 * 4096), (9, 911 * 4096 + 5)])
def test_update_all_gather_on_both_sides_of_its_split(P, n):
    """From 5 replicas and 17 M copied elements on (beyond 16 replicas from 0.92 M elements), in tiles that are mostly full, the
    call launches the update and the all-gather; native/launch_rules.cpp pins these sizes to their sides."""
    say("case: update + all-gather, P=%d, %d elements" % (P, n))
    pair = Pair(small_workload([n, 33], P, 0))
    pair.run(iterations=1, fused_gather=True)
    pair.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("P,width,gather", [(1, 0, False), (3, 0, True), (9, 0, False), (9, 2, False), (17, 2, True)])
def test_every_alignment_of_a_runs_ends(P, width, gather, dtype):
    """Runs that begin and end at every element of a 16-byte vector, within one vector, in the
    first, middle and last part of a tile: edge elements have lanes of their own in every kernel."""
    say("case: run ends, P=%d, width %d, gather %s, %s" % (P, width, gather, dtype))
    sizes = list(range(1, 19)) + [4096 + k for k in range(9)] + [1024 * k + k for k in range(1, 8)] + [2047, 2049, 3]
    pair = Pair(small_workload(sizes, P, 40_000, dtype))
    pair.run(iterations=2, width=width, fused_gather=gather)
    if not gather:
        pair.run(iterations=1, width=width, fused=True)
        pair.run(iterations=1, width=width, route="iteration")
    pair.close()


@pytest.mark.parametrize("dtype,P,n", [("f32", 4, 31_300_000), ("f32", 13, 7_800_000), ("f32", 32, 3_200_000),
                                       ("bf16", 5, 16_100_000), ("bf16", 8, 31_300_000), ("bf16", 12, 20_900_000),
                                       ("bf16", 17, 14_800_000)])
def test_launches_with_few_resident_workgroups(dtype, P, n):
    """Long launches, which bound the workgroups per CU, with few and many replicas in each type."""
    say("case: few resident workgroups, %s, P=%d, %d elements" % (dtype, P, n))
    pair = Pair(small_workload([n - 77, 77], P, W.NO_LIMIT, dtype))
    for route in ("calls", "iteration"):
        for fused in (False, True):
            pair.run(iterations=1, route=route, fused=fused)
    pair.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_short_runs(dtype):
    """Thousands of tensors far shorter than a tile in one launch: as many workgroups as fit."""
    say("case: 6000 short tensors, %s" % dtype)
    pair = Pair(small_workload([64, 200, 701] * 2000, 12, W.NO_LIMIT, dtype))
    pair.run(iterations=1)
    pair.run(iterations=1, fused=True)
    pair.close()


@pytest.mark.parametrize("starts", [(0, 0, 0), (4, 4, 4), (28, 28, 28), (0, 12, 20), (16, 4, 28)])
@pytest.mark.parametrize("workers", [(0, 3), (1, 2)])
def test_all_gather_cuts_at_lines(starts, workers):
    """Replicas whose tensors start 16-byte aligned at different places of a 128-byte line, alike or not:
    the cuts of long runs move with them.  One plan has a run whose first tile is shorter than a line, the
    last layer's runs are short; elements around the tensors stay as they are."""
    import paper_2302_12445_amd as dear
    say("case: all-gather, tensors at %s of a line, workers %s" % (starts, workers))
    for x in (5, 3433):  # with 3433 elements in front, the big layer's second run starts 9 elements before a tile's end
        sizes, P = [400_003, x], 3
        op = oracle.plan(sizes, P, W.NO_LIMIT, 4)
        plan = dear.dear_plan(sizes, P, W.NO_LIMIT, 4)
        big = [torch.full((400_100,), 7.0, device=DEV) for _ in range(P)]
        small = [torch.full((x + 64,), 7.0, device=DEV) for _ in range(P)]
        ptrs = [q for p in range(P) for q in (big[p].data_ptr() + 4 * starts[p], small[p].data_ptr() + 4 * starts[p])]
        ctx = dear.dear_ctx_create(plan, dear.DEAR_F32, ptrs, ptrs)
        shards = torch.randn(P, op.total_shard_len, generator=torch.Generator().manual_seed(x))
        dev = shards.to(DEV)
        dear.dear_all_gather_workers(ctx, -1, dev.data_ptr(), workers[0], workers[1])
        torch.cuda.synchronize()
        params = [[np.full(n, 7.0, np.float32) for n in sizes] for _ in range(P)]
        oracle.all_gather(op, -1, shards.numpy(), params, workers=range(workers[0], workers[0] + workers[1]))
        for p in range(P):
            for got, want in ((big[p], params[p][0]), (small[p], params[p][1])):
                full = np.full(got.numel(), 7.0, np.float32)
                full[starts[p]:starts[p] + want.size] = want
                assert np.array_equal(_bits(got.cpu().numpy()), _bits(full)), (x, p)
        ctx.destroy()


def test_calls_beyond_the_largest_all_gather():
    """From 2^24 workgroups on an all-gather cannot be launched: dear_all_gather and dear_iteration refuse it and
    leave everything as it was, dear_update_all_gather takes such a call in its one kernel, a bounded grid
    takes it anyway.  1024 replicas that share their tensors stand for a card full of them."""
    import paper_2302_12445_amd as dear
    from paper_2302_12445_amd import binding
    n, P = 4104 * 4096, 1024
    say("case: 2^24 workgroups, %d elements, P=%d in one set of tensors" % (n, P))
    plan, op = dear.dear_plan([n], P, W.NO_LIMIT, 4), oracle.plan([n], P, W.NO_LIMIT, 4)
    gen = torch.Generator(device=DEV).manual_seed(5)
    grad, param = torch.zeros(n, device=DEV), torch.full((n,), 7.0, device=DEV)
    ctx = dear.dear_ctx_create(plan, dear.DEAR_F32, [grad.data_ptr()] * P, [param.data_ptr()] * P)
    assert 4 * P * len(dear.dear_plan_tiles(plan)[0]) >= 1 << 24
    g, w, v = (torch.empty(P, op.total_shard_len, device=DEV).normal_(0.0, 1.0, generator=gen) for _ in range(3))
    ref = [t.cpu().numpy().copy() for t in (g, w, v)]
    with pytest.raises(dear.DearError) as e:
        dear.dear_all_gather(ctx, -1, w.data_ptr())
    assert e.value.status == binding.DEAR_EINVAL
    with pytest.raises(dear.DearError) as e:
        dear.dear_iteration(ctx, -1, g.data_ptr(), w.data_ptr(), v.data_ptr(), 0.1, 0.9)
    assert e.value.status == binding.DEAR_EINVAL
    torch.cuda.synchronize()
    for t, r in zip((g, w, v), ref):
        assert np.array_equal(_bits(t.cpu().numpy()), _bits(r))
    assert bool((param == 7.0).all())

    dear.dear_update_all_gather(ctx, -1, g.data_ptr(), w.data_ptr(), v.data_ptr(), 0.1, 0.9)
    torch.cuda.synchronize()
    oracle.shard_update(op, -1, ref[0], ref[1], ref[2], 0.1, 0.9)
    host = [[np.zeros(n, np.float32)]] * P
    oracle.all_gather(op, -1, ref[1], host, workers=range(0, 1))
    assert np.array_equal(_bits(w.cpu().numpy()), _bits(ref[1])) and np.array_equal(_bits(v.cpu().numpy()), _bits(ref[2]))
    assert np.array_equal(_bits(param.cpu().numpy()), _bits(host[0][0]))

    param.fill_(7.0)
    dear.dear_ctx_set_max_workgroups(ctx, 256)
    dear.dear_all_gather(ctx, -1, w.data_ptr())
    torch.cuda.synchronize()
    assert np.array_equal(_bits(param.cpu().numpy()), _bits(host[0][0]))
    ctx.destroy()
