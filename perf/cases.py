"""Performance cases of the gradient-aggregation path: what a user of the framework has it do,
through the public entry points, from calls where only launches count to ones that stream tens
of gigabytes, in both gradient types and every way the framework offers to run an iteration.

listed() and draw() give cases (dicts of plain values); prepare() builds what a training program
holds before the call; run() is one pass; work() the traffic and arithmetic a pass cannot do
without; tolerance() how far another correct implementation may be off; exact() the result in 64
bits from plain torch operations.

Paths (case["path"]):
  step       EmulatedWorkers.iteration: reduce-scatter, update, all-gather
  fused      the same with fused_update (what the schedule and DistOptim launch by default)
  gather     the same with fused_gather
  graph      one iteration captured once into a HIP graph, a pass replays it
  calls      the C-ABI entry points called bucket by bucket (or once for all buckets) on tensors that
             the program allocated itself, 16-byte aligned and no more
  static     dear_reduce_scatter_static, the entry point that allocates nothing
  replan     EmulatedWorkers.replan: change of the buffer size with the optimizer state carried over
  schedule   iterations of DearSchedule: aggregation beside compute on a second stream
  dist       a training step of P module replicas under DistOptim
"""
from __future__ import annotations

import math
import random

import torch

import paper_2302_12445_amd as dear
from paper_2302_12445_amd.dist_optim import DistOptim
from paper_2302_12445_amd.emulation import EmulatedWorkers
from paper_2302_12445_amd.schedule import DearSchedule

DEV = "cuda:0"
KB, MB = 1 << 10, 1 << 20
LR, MU = 0.1, 0.9
EMULATED = ("step", "fused", "gather", "graph", "replan", "schedule")
SCHEDULE_ITERATIONS = 2


# ------------------------------------------------------------------------------------ the cases
def _case(path, sizes, P, grad, threshold, launch="bucket", **more):
    return dict({"path": path, "sizes": sizes, "P": P, "grad": grad, "threshold": threshold, "launch": launch}, **more)


def listed():
    return [
        # eight small tensors in five buckets: everything sits in caches, launches and latency count
        dict(_case("step", "tiny", 4, "f32", 256 * KB), name="tiny_step"),
        # the same, recorded once as a launch-bound program does
        dict(_case("graph", "tiny", 4, "f32", 256 * KB), name="tiny_graph"),
        # a convolutional net's 161 tensors at the default 25 MB buffer: launches of 10 to 40 us
        dict(_case("step", "resnet50", 8, "f32", 25 * MB), name="resnet50_step"),
        # many ragged tensors, an odd number of workers, bf16, tensors of the program's own
        dict(_case("calls", "ragged", 7, "bf16", 25 * MB, layers=604, elems=20_013_929, fused=True), name="ragged_bf16_p7"),
        # 64 workers, one launch per phase: the widest reduction
        dict(_case("calls", "resnet50", 64, "f32", 16 * MB, launch="all", fused=False), name="resnet50_p64_all"),
        # a transformer with the update moved behind the all-gather's launch
        dict(_case("gather", "bert_base", 16, "f32", 64 * MB), name="bert_base_gather"),
        # the default benchmark: the three phases of the largest model
        dict(_case("step", "bert_large", 8, "bf16", 64 * MB), name="bert_large_step"),
        # what BackPipe launches: reduce-scatter and update in one kernel
        dict(_case("fused", "bert_large", 8, "bf16", 64 * MB), name="bert_large_fused"),
        # a program that may not allocate: tables go up with each call
        dict(_case("static", "resnet50", 8, "f32", 25 * MB, launch="all"), name="resnet50_static"),
        # one trial of the buffer-size tuner: new plan, parameters and momentum re-sharded
        dict(_case("replan", "bert_base", 8, "f32", 64 * MB, other=25 * MB), name="bert_base_replan"),
        # the aggregation beside compute, as the schedule issues it (bounded grids)
        dict(_case("schedule", "bert_base", 16, "f32", 64 * MB, gemm=2048, ff=4, bp=8), name="bert_base_schedule"),
        # a training step driven by autograd hooks
        dict(_case("dist", "mlp", 4, "f32", 4 * MB, width=512, hidden=2048, blocks=3, batch=32), name="dist_mlp"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the ranges above: ragged tensor lists from the tiny one's size to a few hundred
    megabytes a worker, 2 to 64 workers, buffers from no fusion to no limit, every path."""
    path = rng.choice(["step", "step", "fused", "fused", "gather", "calls", "calls", "static", "graph", "replan", "dist"])
    if path == "dist":
        return _case("dist", "mlp", rng.randint(2, 4), "f32", _log_uniform(rng, 64 * KB, 16 * MB), width=_log_uniform(rng, 33, 700),
                     hidden=_log_uniform(rng, 64, 2500), blocks=rng.randint(1, 3), batch=rng.randint(5, 64))
    grad = rng.choice(["f32", "bf16"])
    g = 4 if grad == "f32" else 2
    P = rng.choice([2, 3, 4, 5, 6, 7, 8, 8, 8, 11, 12, 16, 16, 24, 32] + ([48, 64] if path in ("calls", "static") else []))
    layers = _log_uniform(rng, 6, 600)
    elems = _log_uniform(rng, max(200_000, 50 * layers), min(110_000_000, int(14e9 / (P * (g + 4)))))
    threshold = rng.choice([0, -1] + [_log_uniform(rng, 256 * KB, 64 * MB)] * 8)  # -1: no limit
    if threshold == 0 and layers > 100:
        threshold = 25 * MB
    launch = "all" if path == "static" else rng.choice(["bucket", "bucket", "all"])
    more = {"layers": layers, "elems": elems}
    if path == "calls":
        more["fused"] = rng.random() < 0.5
    if path == "replan":
        more["other"] = _log_uniform(rng, 256 * KB, 64 * MB)
    return _case(path, "ragged", P, grad, threshold, launch=launch, **more)


# ------------------------------------------------------------------------------------ tensor lists
def _resnet50():
    s = [64 * 3 * 49, 64, 64]
    wide = 64
    for planes, blocks in ((64, 3), (128, 4), (256, 6), (512, 3)):
        for blk in range(blocks):
            s += [planes * wide, planes, planes, planes * planes * 9, planes, planes, planes * planes * 4, planes * 4, planes * 4]
            if blk == 0:
                s += [planes * 4 * wide, planes * 4, planes * 4]
            wide = planes * 4
    return s + [1000 * 2048, 1000]


def _bert(layers, h, ffn):
    s = [30522 * h, 512 * h, 2 * h, h, h]
    for _ in range(layers):
        s += [h * h, h] * 4 + [h, h, h * ffn, ffn, ffn * h, h, h, h]
    return s + [h * h, h, h * h, h, h, h, 30522, 2 * h, 2]


def _ragged(layers, elems):
    """A weight followed by two vectors, over and over: weights of very different and mostly odd
    sizes, about `elems` elements in all.  The same list for the same two numbers."""
    rng = random.Random(layers * 1_000_003 + elems)
    raw = [math.exp(rng.gauss(0.0, 1.2)) if l % 3 == 0 else 0.0 for l in range(layers)]
    vec = [0 if l % 3 == 0 else rng.choice([1, 2, 10, 33, 64, 127, 256, 512, 1000]) for l in range(layers)]
    scale = max(1.0, elems - sum(vec)) / sum(raw)
    return [max(1, int(r * scale)) if r else v for r, v in zip(raw, vec)]


def _mlp(case):
    s = []
    for _ in range(case["blocks"]):
        s += [case["hidden"] * case["width"], case["hidden"], case["width"] * case["hidden"], case["width"]]
    return s


def _sizes(case):
    kind = case["sizes"]
    if kind == "tiny":
        return [4096, 64, 65536, 128, 262144, 256, 16384, 10]
    if kind == "resnet50":
        return _resnet50()
    if kind == "bert_base":
        return _bert(12, 768, 3072)
    if kind == "bert_large":
        return _bert(24, 1024, 4096)
    if kind == "mlp":
        return _mlp(case)
    return _ragged(case["layers"], case["elems"])


def _g(case):
    return 4 if case["grad"] == "f32" else 2


def _dtype(case):
    return torch.float32 if case["grad"] == "f32" else torch.bfloat16


def _threshold(bytes_):
    return dear.DEAR_NO_LIMIT if bytes_ < 0 else bytes_


# ------------------------------------------------------------------------------------ inputs
def _starts(case, sizes, elem_bytes):
    """Where each layer starts in a replica's one buffer, and the buffer's length: 256-byte
    boundaries as EmulatedWorkers lays them out, 16-byte ones for the program's own tensors."""
    a = (256 if case["path"] in EMULATED else 16) // elem_bytes
    starts, pos = [], 0
    for n in sizes:
        starts.append(pos)
        pos = (pos + n + a - 1) // a * a
    return starts, pos


def _rng(seed, what):
    return torch.Generator(device=DEV).manual_seed(seed * 7919 + what)


def _grad_buffer(case, sizes, seed, p):
    """Worker p's gradients, all layers in one buffer: N(0, 1e-3)."""
    buf = torch.empty(_starts(case, sizes, _g(case))[1], dtype=_dtype(case), device=DEV)
    return buf.normal_(0.0, 1e-3, generator=_rng(seed, p))


def _param_buffer(case, sizes, seed):
    buf = torch.empty(_starts(case, sizes, 4)[1], dtype=torch.float32, device=DEV)
    return buf.uniform_(-0.1, 0.1, generator=_rng(seed, 1001))


def _momentum(shape, seed):
    return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(0.0, 1e-3, generator=_rng(seed, 1002))


def _layers_of(buf, starts, sizes):
    return [buf[s:s + n] for s, n in zip(starts, sizes)]


def _batch(case, seed):
    n = case["P"] * case["batch"]
    x = torch.randn(n, case["width"], device=DEV, generator=_rng(seed, 1003))
    y = torch.randn(n, case["width"], device=DEV, generator=_rng(seed, 1004))
    return x.view(case["P"], case["batch"], -1), y.view(case["P"], case["batch"], -1)


def _module(case, seed, dtype=torch.float32):
    """Linear / ReLU blocks; weights from the seed alone."""
    mods, gen = [], _rng(seed, 1005)
    for _ in range(case["blocks"]):
        mods += [torch.nn.Linear(case["width"], case["hidden"], device=DEV), torch.nn.ReLU(),
                 torch.nn.Linear(case["hidden"], case["width"], device=DEV)]
    net = torch.nn.Sequential(*mods)
    with torch.no_grad():
        for p in net.parameters():
            p.normal_(0.0, 0.02, generator=gen)
    return net.to(dtype)


class _State:
    pass


def _prepare_emulated(case, seed, st):
    sizes = _sizes(case)
    em = EmulatedWorkers(sizes, case["P"], case["grad"], _threshold(case["threshold"]), DEV)
    st.em = em
    st.param_buffers = [rep[0]._base for rep in em.params]
    for p in range(case["P"]):
        em.grads[p][0]._base.copy_(_grad_buffer(case, sizes, seed, p))
    if case["path"] == "replan":  # momentum as training leaves it: padding slots hold zeros
        mom = _momentum(st.param_buffers[0].shape, seed)
        st.param_buffers[0].copy_(mom)
        dear.dear_scatter_params(em.ctx, 0, em.shard_mom.data_ptr(), torch.cuda.current_stream().cuda_stream)
    else:
        em.shard_mom.copy_(_momentum(em.shard_mom.shape, seed))
    param = _param_buffer(case, sizes, seed)
    for buf in st.param_buffers:
        buf.copy_(param)
    em.scatter_params(0)
    if case["path"] == "graph":
        st.graph = em.capture_iteration(LR, MU, per_bucket=case["launch"] == "bucket")
    if case["path"] == "schedule":
        st.sched = DearSchedule(em, LR, MU, gemm_dim=case["gemm"], ff_gemms=case["ff"], bp_gemms=case["bp"])
    if case["path"] == "replan":
        st.next = [_threshold(case["other"]), _threshold(case["threshold"])]


def _prepare_calls(case, seed, st):
    sizes, P = _sizes(case), case["P"]
    st.plan = dear.dear_plan(sizes, P, _threshold(case["threshold"]), _g(case))
    gs, glen = _starts(case, sizes, _g(case))
    st.grads = torch.empty(P, (glen + 127) // 128 * 128, dtype=_dtype(case), device=DEV)
    for p in range(P):
        st.grads[p, :glen] = _grad_buffer(case, sizes, seed, p)
    st.grad_ptrs = [st.grads[p].data_ptr() + s * _g(case) for p in range(P) for s in gs]
    st.dtype = dear.DEAR_F32 if case["grad"] == "f32" else dear.DEAR_BF16
    st.shard_grad = torch.zeros(P, st.plan.total_shard_len, device=DEV)
    st.buckets = [-1] if case["launch"] == "all" else list(range(st.plan.n_buckets))
    if case["path"] == "static":
        return
    ps = _starts(case, sizes, 4)[0]
    st.params = _param_buffer(case, sizes, seed).expand(P, -1).contiguous()
    param_ptrs = [st.params[p].data_ptr() + 4 * s for p in range(P) for s in ps]
    st.ctx = dear.dear_ctx_create(st.plan, st.dtype, st.grad_ptrs, param_ptrs)
    st.shard_param = torch.zeros_like(st.shard_grad)
    st.shard_mom = _momentum(st.shard_grad.shape, seed)
    dear.dear_scatter_params(st.ctx, 0, st.shard_param.data_ptr(), torch.cuda.current_stream().cuda_stream)


def _prepare_dist(case, seed, st):
    st.models = [_module(case, seed) for _ in range(case["P"])]
    st.x, st.y = _batch(case, seed)
    st.opt = DistOptim(st.models, lr=LR, momentum=MU, fusion_threshold_bytes=_threshold(case["threshold"]))


def prepare(case, seed):
    st = _State()
    st.case = case
    if case["path"] in EMULATED:
        _prepare_emulated(case, seed, st)
    elif case["path"] == "dist":
        _prepare_dist(case, seed, st)
    else:
        _prepare_calls(case, seed, st)
    return st


# ------------------------------------------------------------------------------------ one pass
def _run_calls(st):
    h = torch.cuda.current_stream().cuda_stream
    g, w, v = st.shard_grad.data_ptr(), st.shard_param.data_ptr(), st.shard_mom.data_ptr()
    if st.case["fused"]:
        for b in st.buckets:
            dear.dear_reduce_scatter_update(st.ctx, b, w, v, LR, MU, h)
    else:
        for b in st.buckets:
            dear.dear_reduce_scatter(st.ctx, b, g, h)
            dear.dear_shard_update(st.ctx, b, g, w, v, LR, MU, h)
    for b in reversed(st.buckets):
        dear.dear_all_gather(st.ctx, b, w, h)
    return {"w": st.shard_param, "v": st.shard_mom, "params": st.params, "g": None if st.case["fused"] else st.shard_grad}


def run(st):
    path = st.case["path"]
    if path == "calls":
        return _run_calls(st)
    if path == "static":
        for b in st.buckets:
            dear.dear_reduce_scatter_static(st.plan, st.dtype, st.grad_ptrs, b, st.shard_grad.data_ptr(),
                                            torch.cuda.current_stream().cuda_stream)
        return {"g": st.shard_grad}
    if path == "dist":
        for p, model in enumerate(st.models):
            torch.nn.functional.mse_loss(model(st.x[p]), st.y[p]).backward()
        st.opt.step()
        return {"w": st.opt.shard_param, "v": st.opt.shard_mom, "params": [[q.detach() for q in m.parameters()] for m in st.models]}
    em = st.em
    if path == "replan":
        st.next.reverse()
        em.replan(threshold_bytes=st.next[1])
        return {"w": em.shard_param, "v": em.shard_mom, "params": st.param_buffers[:1]}
    if path == "graph":
        st.graph.replay()
    elif path == "schedule":
        here = torch.cuda.current_stream()
        for s in (st.sched.compute, st.sched.comm):
            s.wait_stream(here)
        for _ in range(SCHEDULE_ITERATIONS):
            st.sched.iteration("dear")
        for s in (st.sched.compute, st.sched.comm):
            here.wait_stream(s)
    else:
        em.iteration(LR, MU, per_bucket=st.case["launch"] == "bucket", fused_update=path == "fused", fused_gather=path == "gather")
    keeps_g = path in ("step", "graph", "gather")
    return {"w": em.shard_param, "v": em.shard_mom, "params": st.param_buffers, "g": em.shard_grad if keeps_g else None}


# ------------------------------------------------------------------------------------ what a pass needs
def work(case):
    """Each gradient, shard and parameter read once where it is an input and written once where it
    is an output; one addition per worker and element, one product for the mean, four for the update."""
    N, P, g, path = sum(_sizes(case)), case["P"], _g(case), case["path"]
    if path == "static":
        return {"bytes": N * (g * P + 4), "flops": N * P}
    if path == "replan":
        return {"bytes": N * 16, "flops": 0}
    keeps_g = path in ("step", "graph", "gather") or (path == "calls" and not case["fused"])
    bytes_, flops = N * (g * P + 4 * P + 16 + (4 if keeps_g else 0)), N * (P + 4)
    if path == "schedule":
        buckets = len(_plan(_sizes(case), P, case["threshold"], g))
        gemms, dim = buckets * (case["ff"] + case["bp"]), case["gemm"]
        return {"bytes": SCHEDULE_ITERATIONS * (bytes_ + gemms * 12 * dim * dim),
                "flops": SCHEDULE_ITERATIONS * (flops + gemms * 2 * dim ** 3)}
    if path == "dist":  # each replica reads its weights forward and backward and writes its gradients
        return {"bytes": bytes_ + 12 * N * P, "flops": flops + 6 * N * case["batch"] * P}
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    """The sums have a fixed order and every operation a rounding of its own, so the outputs have one
    right value; only a training step has library products in it, whose sums may be ordered otherwise."""
    return {"rel": 1e-5} if case["path"] == "dist" else "exact"


# ------------------------------------------------------------------------------------ 64 bits
def _plan(sizes, P, threshold, g):
    """[(layers in packing order, elements, shard length)] of each bucket: layers from the last on,
    a bucket closed before the layer that would take it past the threshold."""
    limit = math.inf if threshold < 0 else threshold // g
    groups = []
    for l in reversed(range(len(sizes))):
        if groups and sum(sizes[i] for i in groups[-1]) + sizes[l] <= limit:
            groups[-1].append(l)
        else:
            groups.append([l])
    out = []
    for ls in groups:
        d = sum(sizes[l] for l in ls)
        out.append((ls, d, (-(-d // P) + 31) // 32 * 32))
    return out


def _to_shards(layers, plan, P):
    rows = []
    for ls, d, S in plan:
        flat = torch.zeros(P * S, dtype=torch.float64, device=DEV)
        flat[:d] = torch.cat([layers[l] for l in ls])
        rows.append(flat.view(P, S))
    return torch.cat(rows, 1)


def _from_shards(shards, plan, layers):
    at = 0
    for ls, d, S in plan:
        flat = shards[:, at:at + S].reshape(-1)
        at += S
        pos = 0
        for l in ls:
            n = layers[l].numel()
            layers[l].copy_(flat[pos:pos + n])
            pos += n


def _exact_dist(case, seed):
    net = _module(case, seed, torch.float64)
    x, y = _batch(case, seed)
    loss = sum(torch.nn.functional.mse_loss(net(a.double()), b.double()) for a, b in zip(x, y)) / case["P"]
    loss.backward()
    params = [p.detach() - LR * p.grad for p in net.parameters()]
    plan = _plan(_sizes(case), case["P"], case["threshold"], 4)
    return {"w": _to_shards([p.reshape(-1) for p in params], plan, case["P"]),
            "v": _to_shards([p.grad.reshape(-1) for p in net.parameters()], plan, case["P"]),
            "params": [params for _ in range(case["P"])]}


def exact(case, seed):
    path = case["path"]
    if path == "dist":
        return _exact_dist(case, seed)
    sizes, P = _sizes(case), case["P"]
    param = _param_buffer(case, sizes, seed).double()
    layers = _layers_of(param, _starts(case, sizes, 4)[0], sizes)
    if path == "replan":  # the first pass goes to the other threshold
        plan = _plan(sizes, P, case["other"], _g(case))
        mom = _layers_of(_momentum(param.shape, seed).double(), _starts(case, sizes, 4)[0], sizes)
        return {"w": _to_shards(layers, plan, P), "v": _to_shards(mom, plan, P), "params": [param]}
    plan = _plan(sizes, P, case["threshold"], _g(case))
    total = None
    for p in range(P):
        x = _grad_buffer(case, sizes, seed, p).double()
        total = x if total is None else total.add_(x)
    mean = _to_shards([t / P for t in _layers_of(total, _starts(case, sizes, _g(case))[0], sizes)], plan, P)
    if path == "static":
        return {"g": mean}
    w = _to_shards(layers, plan, P)
    v = _momentum(w.shape, seed).double()
    for _ in range(SCHEDULE_ITERATIONS if path == "schedule" else 1):
        v = MU * v + mean
        w = w - LR * v
    _from_shards(w, plan, layers)
    params = param.expand(P, -1) if path == "calls" else [param] * P
    keeps_g = path in ("step", "graph", "gather") or (path == "calls" and not case["fused"])
    return {"w": w, "v": v, "params": params, "g": mean if keeps_g else None}
