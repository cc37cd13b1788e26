"""Performance cases of the fused local update + P-Reduce path.

A case is one training step's synchronization (or one replay of a captured
period of steps) as a program that trains N replicas on one GPU runs it: the
buffers are registered once (``Replicas``), then every pass is one call through
the Python binding.  The sizes come from the repository's workloads, tests and
smoke run (seedgen/workloads.py, __graft_entry__.py), or are generic.

A case's fields:
  entry     "step" (group generation and the fused launch, ``rip_step``),
            "preduce" (``rip_preduce`` with the program's own groups), "local"
            (``rip_local_step``), "average" (pure P-Reduce, no update) or
            "graph" (a HIP graph of one period of fused steps, replayed)
  n         replicas
  params    elements of a replica registered as one flat buffer, or 0: the
            layer tensors of ``net`` ("resnet50", "vgg16", or "plain" with
            ``depth`` and ``width``)
  separate  the layer tensors are buffers of their own (false: views back to
            back in one flat buffer per replica)
  dtype     "f32" or "bf16" storage
  momentum, decay, nesterov   the optimizer (0, 0 and False: plain SGD)
  sizes     sizes of the step's groups; replicas outside them update alone
  idle      how many of the grouped replicas do not update this step (they
            only average, as a straggler's group members do)

Every pass takes the next of four seeded group rows, as a periodic schedule
does.  The updated parameters (and momenta) are the outputs.
"""
import random

import numpy as np
import torch

import paper_1909_08029_amd as rip
from seedgen.workloads import RESNET50_PARAMS, VGG16_SEGMENTS

PERIOD = 4  # rows of the periodic schedule (the paper's static schedules have four)


def _case(name, entry, n, params, sizes, dtype="f32", momentum=0.0, decay=0.0, nesterov=False,
          idle=0, net="", depth=0, width=0, separate=False):
    case = dict(entry=entry, n=n, params=params, net=net, depth=depth, width=width,
                separate=separate, dtype=dtype, momentum=momentum, decay=decay,
                nesterov=nesterov, sizes=",".join(str(k) for k in sizes), idle=idle)
    return dict(case, name=name) if name else case


def listed():
    return [
        # the smallest call: the smoke run's four small replicas, a group of
        # three and a lone update; latency of one call
        _case("smoke_4x12k", "preduce", 4, 12293, [3]),
        # the small workload: 1M parameters, a fixed group, scheduled and
        # launched in one call
        _case("step_4x1m", "step", 4, 1_048_576, [3]),
        # a captured period of steps over small bf16 replicas, as a loop that
        # is launch-bound replays it (odd size, lone updates beside a group)
        _case("graph_8x262k_bf16_mom", "graph", 8, 262_147, [3, 2], "bf16", 0.9),
        # a small network kept as separate layer tensors (weights, scale and
        # shift vectors; odd sizes), the paper's ResNet optimizer settings
        _case("layers_16_plain_mom_wd", "step", 16, 0, [4, 4, 4, 4], momentum=0.9, decay=1e-4,
              net="plain", depth=19, width=17, separate=True),
        # pure averaging of an odd, ordinary size in groups of three
        _case("average_12x3m", "average", 12, 3_000_001, [3, 3, 3, 3]),
        # All-Reduce as one group of the most replicas a handle takes
        _case("allreduce_256x65k_bf16", "preduce", 256, 65_539, [256], "bf16"),
        # the local update alone (the unfused form's first pass), bf16, with
        # Nesterov momentum and weight decay
        _case("local_8x10m_bf16_nesterov", "local", 8, 10_000_019, [], "bf16", 0.9, 1e-4, True),
        # ResNet-50's 161 tensors as separate buffers on 16 replicas, with the
        # paper's optimizer for it
        _case("layers_16_resnet50_mom_wd", "step", 16, 0, [4, 4, 4, 4], momentum=0.9, decay=1e-4,
              net="resnet50", separate=True),
        # 32 heterogeneous replicas divided into groups of two to eight, some
        # of whose members (a straggler's) do not update this step
        _case("hetero_32x25m", "preduce", 32, RESNET50_PARAMS, [2, 7, 4, 8, 3, 5, 2], idle=4),
        # All-Reduce of 32 replicas of ResNet-50's size
        _case("allreduce_32x25m", "preduce", 32, RESNET50_PARAMS, [32]),
        # VGG-16 on 16 replicas with momentum, static groups of eight
        _case("step_16_vgg16_mom", "step", 16, 0, [8, 8], momentum=0.9, net="vgg16"),
        # the largest workload: eight bf16 replicas of 1.3G parameters
        _case("step_8x1300m_bf16", "step", 8, 1_300_000_000, [4, 4], "bf16"),
    ]


def _equal_sizes(n, k):
    return [k] * (n // k)


def draw(rng):
    entry = rng.choice(["step", "step", "preduce", "preduce", "local", "average", "graph"])
    dtype = rng.choice(["f32", "bf16"])
    n = min(256, max(2, int(2 ** rng.uniform(1, 6.5))))
    top = 33 if entry != "graph" else 26  # bytes of parameters over all replicas
    total = 2 ** rng.uniform(16, top)
    per = max(256, int(total / n / (2 if dtype == "bf16" else 4)))
    style = rng.choice(["fours", "pairs", "mixed", "mixed", "eights", "threes", "all"])
    if entry == "local":
        sizes = []
    elif style == "all":
        sizes = [n]
    elif style == "mixed":  # a random division, the rest update alone
        sizes, left = [], n
        while left > 1:
            k = min(left, rng.randint(2, 8))
            sizes.append(k)
            left -= k
            if rng.random() < 0.1:
                break
    else:
        sizes = _equal_sizes(n, {"pairs": 2, "threes": 3, "fours": 4, "eights": 8}[style])
        sizes = sizes or [n]
    momentum = 0.0 if entry == "average" else rng.choice([0.0, 0.0, 0.9])
    decay = 0.0 if entry == "average" else rng.choice([0.0, 0.0, 1e-4])
    nesterov = bool(momentum) and rng.random() < 0.25
    idle = rng.randint(1, max(1, sum(sizes) // 4)) if entry == "preduce" and rng.random() < 0.4 else 0
    if per > 60_000 and rng.random() < 0.35:  # separate layer tensors, about `per` elements
        depth = rng.randint(6, 48)
        width = max(3, int((per / (9 * 7 * depth)) ** 0.5))
        return _case("", entry, n, 0, sizes, dtype, momentum, decay, nesterov, idle, "plain",
                     depth, width, True)
    return _case("", entry, n, per | (rng.random() < 0.6), sizes, dtype, momentum, decay,
                 nesterov, idle)


# ---------------------------------------------------------------------------
def _plain_net(depth, width):
    """A stack of 3x3 convolutions with a scale and a shift vector each, the
    width doubled after each third, and a ten-way head."""
    out, c = [27 * width, width, width], width
    for i in range(1, depth):
        d = width << min(2, 3 * i // depth)
        out += [9 * c * d, d, d]
        c = d
    return out + [10 * c, 10]


def _resnet50():
    """The tensors of ResNet-50 (ImageNet): convolutions and their batch
    norms' scales and shifts, then the classifier; 25,557,032 in total."""
    out, c = [64 * 3 * 49, 64, 64], 64
    for width, blocks in ((64, 3), (128, 4), (256, 6), (512, 3)):
        for b in range(blocks):
            out += [c * width, width, width, width * width * 9, width, width,
                    width * width * 4, width * 4, width * 4]
            if b == 0:
                out += [c * width * 4, width * 4, width * 4]
            c = width * 4
    return out + [2048 * 1000, 1000]


def _segments(case):
    if case["params"]:
        return [int(case["params"])]
    if case["net"] == "resnet50":
        return _resnet50()
    if case["net"] == "vgg16":
        return list(VGG16_SEGMENTS)
    return _plain_net(case["depth"], case["width"])


def _sizes(case):
    return [int(k) for k in case["sizes"].split(",") if k]


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _layout(case):
    """Element offset of each segment within a replica's buffer and the
    buffer's length: back to back, or each at its own 512-byte boundary."""
    per = 512 // (2 if case["dtype"] == "bf16" else 4)
    offs, end = [], 0
    for m in _segments(case):
        if case["separate"]:
            end = -(-end // per) * per
        offs.append(end)
        end += m
    return offs, -(-end // per) * per


def _rows(case, seed):
    """PERIOD rows of (active, groups): seeded partitions of the replicas."""
    rng, n, rows = random.Random(seed), case["n"], []
    for _ in range(PERIOD):
        ids = list(range(n))
        rng.shuffle(ids)
        groups, at = [], 0
        for k in _sizes(case):
            groups.append(tuple(sorted(ids[at:at + k])))
            at += k
        idle = set(ids[:case["idle"]])
        active = [] if case["entry"] == "average" else [i for i in range(n) if i not in idle]
        rows.append((active, groups))
    return rows


def _opt(case):
    f = lambda x: float(np.float32(x))  # noqa: E731 -- the library takes fp32 scalars
    return f(0.1 if case["dtype"] == "f32" else 0.01), f(case["momentum"]), f(case["decay"])


def _buffers(case, seed):
    """Parameters, gradients and momenta: one row per replica."""
    n, pitch = case["n"], _layout(case)[1]
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def kind(sigma):
        rows = torch.empty((n, pitch), dtype=_dtype(case), device="cuda")
        if n * pitch < 1 << 28:
            return rows.normal_(0.0, sigma, generator=gen)
        for r in range(n):
            rows[r].normal_(0.0, sigma, generator=gen)
        return rows

    return (kind(1.0), kind(0.01) if case["entry"] != "average" else None,
            kind(0.01) if case["momentum"] else None)


def _outputs(w, v):
    """The updated parameters and momenta; row by row where they are large."""
    whole = w.numel() < 1 << 32
    out = {"param": w if whole else list(w)}
    if v is not None:
        out["mom"] = v if whole else list(v)
    return out


def prepare(case, seed):
    w, g, v = _buffers(case, seed)
    segs, (offs, _) = _segments(case), _layout(case)

    def views(rows):
        return None if rows is None else [[row[o:o + m] for o, m in zip(offs, segs)]
                                          for row in rows]

    lr, mu, wd = _opt(case)
    opt = dict(lr=lr, momentum=mu, weight_decay=wd, nesterov=case["nesterov"])
    s = dict(entry=case["entry"], w=w, g=g, v=v, rows=_rows(case, seed), t=0, opt=opt,
             rep=rip.Replicas(views(w), views(g), views(v)))
    if case["entry"] == "step":
        s["sched"] = rip.Scheduler(case["n"], rip.SCHED_TABLE,
                                   table=[groups for _, groups in s["rows"]])
    if case["entry"] == "graph":
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for active, groups in s["rows"]:
                rip.rip_preduce(s["rep"], groups, active, **opt)
    return s


def run(state):
    entry, t = state["entry"], state["t"]
    state["t"] = t + 1
    if entry == "graph":
        state["graph"].replay()
    elif entry == "step":
        rip.rip_step(state["sched"], state["rep"], t, **state["opt"])
    else:
        active, groups = state["rows"][t % PERIOD]
        if entry == "preduce":
            rip.rip_preduce(state["rep"], groups, active, **state["opt"])
        elif entry == "local":
            rip.rip_local_step(state["rep"], active, **state["opt"])
        else:
            rip.rip_preduce(state["rep"], groups)
    return _outputs(state["w"], state["v"])


def work(case):
    """Every updating replica reads its parameters and gradient (and momentum)
    and writes its parameters (and momentum); a group member that does not
    update reads and writes its parameters."""
    esize, params = (2 if case["dtype"] == "bf16" else 4), sum(_segments(case))
    grouped, mom = sum(_sizes(case)), bool(case["momentum"])
    active = 0 if case["entry"] == "average" else case["n"] - case["idle"]
    only = grouped if case["entry"] == "average" else case["idle"]
    steps = PERIOD if case["entry"] == "graph" else 1
    flops = active * (2 + 2 * mom + 2 * (case["decay"] > 0) + 2 * case["nesterov"])
    flops += sum(k + (k > 1) for k in _sizes(case))
    return {"bytes": steps * params * esize * (active * (5 if mom else 3) + only * 2),
            "flops": steps * params * flops}


def tolerance(case):
    """The order of every fp32 operation and rounding is part of the entry
    points' contract (include/rip.h), so the results are the same bits."""
    return "exact"


def exact(case, seed):
    w, g, v = _buffers(case, seed)
    lr, mu, wd = _opt(case)
    offs, segs = _layout(case)[0], _segments(case)
    spans = list(zip(offs, segs)) if case["separate"] else [(0, sum(segs))]
    rows = _rows(case, seed)[:PERIOD if case["entry"] == "graph" else 1]
    w = [r.double() for r in w]
    v = None if v is None else [r.double() for r in v]

    def update(i, a, b):
        grad = g[i][a:b].double()
        if wd:
            grad += wd * w[i][a:b]
        if v is None:
            w[i][a:b] -= lr * grad
            return
        v[i][a:b] = mu * v[i][a:b] + grad
        w[i][a:b] -= lr * (grad + mu * v[i][a:b] if case["nesterov"] else v[i][a:b])

    for active, groups in rows:
        for o, m in spans:
            for a in range(o, o + m, 1 << 26):
                b = min(o + m, a + (1 << 26))
                for i in active:
                    update(i, a, b)
                for group in groups:
                    mean = sum(w[i][a:b] for i in group) / len(group)
                    for i in group:
                        w[i][a:b] = mean
    if len(w) * len(w[0]) < 1 << 32:
        w, v = torch.stack(w), None if v is None else torch.stack(v)
    return {"param": w} if v is None else {"param": w, "mom": v}
