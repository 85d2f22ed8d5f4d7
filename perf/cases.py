"""The work whose time counts: passes of tenant mixes through `Context.run`, the call a serving program makes per batch.

A case names the tenants (architectures of `synth.zoo`), their storage type, the batch of every tenant, the number of
stages (1 = everything in one stage, more = every operator list cut evenly, the start point of the schedule search),
the way the schedule is issued, the number of streams a stage may use (0 = one per tenant) and whether the compute
units are dealt out between the tenants.

A program that serves keeps its models registered: the context with the weights on the device is made once per case
and shared by the states of that case.  A state is what comes with a request: the images of every tenant, the output
buffers, and a schedule bound to them (a schedule under graph replay belongs to its buffers).
"""
import math

import torch

from paper_2111_14255_amd import api, binding as B
from synth import zoo

# Ways to issue a schedule, as the benchmark and the tests of this repository combine the flags.
FUSED = B.MT_SCHED_FUSE_EXPAND | B.MT_SCHED_FUSE_POOL
MODES = {
    "plain": 0,                                                                    # the paper's: one issuing thread, event barriers
    "fused": FUSED,                                                                # the same with neighbouring operators fused
    "threads": FUSED | B.MT_SCHED_PARALLEL_ISSUE | B.MT_SCHED_HOST_BARRIER,        # the benchmark's mode
    "coissue": FUSED | B.MT_SCHED_PARALLEL_ISSUE | B.MT_SCHED_HOST_BARRIER | B.MT_SCHED_COISSUE,   # its searched schedule's mode
    "counter": FUSED | B.MT_SCHED_PARALLEL_ISSUE | B.MT_SCHED_COUNTER_BARRIER,     # stage barriers by a counter word
    "graph": B.MT_SCHED_GRAPH | FUSED,                                             # whole-schedule replay
    "stream_graphs": B.MT_SCHED_STREAM_GRAPHS | FUSED,                             # replay per stream and stage
}
TINY = ("tinyA", "tinyB", "tinyC", "tinyD")
FULL = ("alexnet", "alexnet_published", "inceptionv3", "mobilenetv2", "resnet18", "resnet34", "resnet50", "resnet101", "vgg16")
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
MAX_MACS = {"f32": 8.8e9, "f16": 5.4e11, "bf16": 5.4e11}    # of one pass, over all tenants


def _case(tenants, dtype, batch, mode, stages=1, streams=0, shares=False, **name):
    return dict(name, tenants=tenants, dtype=dtype, batch=batch, mode=mode, stages=stages, streams=streams, shares=shares)


def listed():
    return [
        # the smallest call: one tiny image classifier asked for one image, alone on the device
        _case("tinyA", "f32", 1, "plain", name="tiny_single_f32"),
        # three tiny tenants in two stages (the smallest of the benchmark's workloads)
        _case("tinyA+tinyB+tinyC", "f32", 1, "plain", stages=2, name="tiny_trio_f32"),
        # one ordinary network, one image: the latency of a single request
        _case("resnet18", "f16", 1, "fused", name="resnet18_latency_f16"),
        # three different networks, one image each, all at once (workload cfg2)
        _case("resnet18+vgg16+mobilenetv2", "f16", 1, "threads", name="trio_b1_f16"),
        # the same under the paper's form: one issuing thread, four stages, event barriers
        _case("resnet18+vgg16+mobilenetv2", "f16", 1, "plain", stages=4, name="trio_b1_staged_f16"),
        # networks of very different depth, replayed as a graph (workload cfg4)
        _case("resnet101+inceptionv3+mobilenetv2+alexnet", "bf16", 1, "graph", name="unbalanced_b1_graph_bf16"),
        # full precision: two networks at a small batch
        _case("resnet18+mobilenetv2", "f32", 4, "threads", name="duo_b4_f32"),
        # an odd batch through the less usual operators: grouped convolution, normalisation, asymmetric windows
        _case("inceptionv3+alexnet_published", "bf16", 5, "counter", stages=3, name="ragged_b5_counter_bf16"),
        # four networks at a small serving batch (workload cfg3)
        _case("resnet18+resnet50+vgg16+mobilenetv2", "f16", 8, "threads", name="quartet_b8_f16"),
        # one network at a throughput batch
        _case("resnet50", "bf16", 64, "plain", name="resnet50_b64_bf16"),
        # eight equal tenants two to a stream (workload cfg5 as its search leaves it)
        _case("+".join(["resnet50"] * 8), "bf16", 16, "coissue", streams=4, name="stress_coissue_bf16"),
        # the same tenants on disjoint eighths of the compute units in eight stages (workload cfg5 as it is stated)
        _case("+".join(["resnet50"] * 8), "bf16", 16, "plain", stages=8, shares=True, name="stress_staged_shares_bf16"),
    ]


def draw(rng):
    """One to five networks (or two to eight equal ones) of any type, at a batch spread over its logarithm, under any mode."""
    while True:
        dtype = rng.choice(("f32", "f16", "f16", "bf16", "bf16"))
        kind = rng.random()
        if kind < 0.15:
            tenants = [rng.choice(TINY) for _ in range(rng.randint(1, 6))]
        elif kind < 0.35:
            tenants = [rng.choice(FULL)] * rng.randint(2, 8)
        else:
            tenants = [rng.choice(FULL) for _ in range(rng.randint(1, 5))]
        batch = max(1, min(64, int(round(2.0 ** rng.uniform(0.0, 6.0)))))
        if sum(zoo.BUILDERS[t](dtype, batch).macs() for t in tenants) > MAX_MACS[dtype]:
            continue
        mode = rng.choice(sorted(MODES))
        stages = 1 if rng.random() < 0.5 else rng.randint(2, 6)
        streams = rng.randint(1, len(tenants)) if rng.random() < 0.5 or mode == "coissue" else 0
        shares = len(tenants) > 1 and mode in ("plain", "fused", "threads") and rng.random() < 0.25
        return _case("+".join(tenants), dtype, batch, mode, stages, streams, shares)


def _specs(case):
    return [zoo.BUILDERS[t](case["dtype"], case["batch"]) for t in case["tenants"].split("+")]


def _params(spec, gen):
    """He-normal filters with the batch norm's scale folded in, small biases: drawn on the device, handed over as arrays."""
    out = []
    for op in spec.ops:
        if op.kind not in ("conv", "dwconv", "fc"):
            out.append(None)
            continue
        h, w, c = op.in_shape
        if op.kind == "conv":
            shape = (op.out_c, op.r, op.s, c // op.groups)
        elif op.kind == "dwconv":
            shape = (c, op.r, op.s)
        else:
            shape = (op.out_c, h * w * c)
        std = math.sqrt(2.0 / math.prod(shape[1:])) * (op.bn_gain if op.bn else 1.0)
        wgt = torch.randn(shape, generator=gen, device="cuda").mul_(std)
        bias = torch.randn(shape[0], generator=gen, device="cuda").mul_(0.1 if op.bn else 0.05)
        out.append({"w": wgt.cpu().numpy(), "bias": bias.cpu().numpy(), "bn": None})
    return out


_server = {}     # the registered models of the case in use: {"key": ..., "ctx": ...}


def _context(case):
    key = (case["tenants"], case["dtype"], case["batch"])
    if _server.get("key") != key:
        _server.clear()
        ctx = api.Context(0)
        for t, spec in enumerate(_specs(case)):
            gen = torch.Generator(device="cuda").manual_seed(7919 * (t + 1))
            model = api.Model(spec, _params(spec, gen))
            ctx.register(model)
            model.close()
        _server.update(key=key, ctx=ctx)
    return _server["ctx"]


def prepare(case, seed):
    ctx = _context(case)
    lens, stages = ctx.lens(), case["stages"]
    pointers = [[-(-n * (j + 1) // stages) for j in range(stages - 1)] for n in lens]
    cus = ctx.device_info().cu_count
    sched = ctx.schedule(pointers, stages, flags=MODES[case["mode"]],
                         concurrency=[case["streams"]] * stages if case["streams"] else None,
                         cu_share=[cus // len(lens)] * len(lens) if case["shares"] else None)
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    inputs = []
    for spec in ctx.specs:
        shape = (spec.batch, spec.in_h, spec.in_w, spec.in_c)
        # tiny networks take pixel values in [0, 1), the others normalised images
        x = (torch.rand if spec.in_h <= 32 else torch.randn)(shape, generator=gen, device="cuda")
        inputs.append(x.to(DTYPES[spec.dtype]))
    outputs = [ctx.make_output(t) for t in range(len(lens))]
    return {"ctx": ctx, "sched": sched, "bound": ctx.bind(inputs, outputs), "outputs": outputs}


def run(state):
    state["ctx"].run(state["sched"], state["bound"])
    return state["outputs"]


def work(case):
    """Images, filters and biases read once, logits written once; the multiply-accumulates of the layers."""
    es = 4 if case["dtype"] == "f32" else 2
    nbytes, flops = 0.0, 0.0
    for spec in _specs(case):
        nbytes += es * spec.batch * (spec.in_h * spec.in_w * spec.in_c + spec.out_features)
        flops += 2.0 * spec.macs()
        for op in spec.ops:
            h, w, c = op.in_shape
            if op.kind == "conv":
                nbytes += es * op.out_c * op.r * op.s * (c // op.groups) + 4 * op.out_c
            elif op.kind == "dwconv":
                nbytes += es * c * op.r * op.s + 4 * c
            elif op.kind == "fc":
                nbytes += es * op.out_c * h * w * c + 4 * op.out_c
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Every layer rounds its result once to the storage type; a chain of up to a hundred layers carries the roundings on."""
    return {"f32": {"rel": 2e-5, "max": 4e-4}, "f16": {"rel": 4e-3, "max": 5e-2}, "bf16": {"rel": 2e-2, "max": 2e-1}}[case["dtype"]]
