"""What a training program asks of this framework, as cases that can be timed.

A program holds K workers' gradients and parameters of one tensor group, either
as per-layer tensors (lists), as K flat buffers ("separate") or interleaved in
one buffer ("tensor"), and in each iteration takes some of these passes:

  step      pack the gradient lists, average them, take the elastic step and
            unpack the workers into the parameter lists: four calls
  pipeline  the same in one call, on the tensor layout
  reduce    the average of K gradients
  easgd     the fused elastic step
  fused     the average and the elastic step in one call
  period    an iteration of the periodic schedule between two exchanges (63 of
            64): plain SGD on every worker
  async     the workers' elastic exchanges with the center, one after the other
  pushpull  synchronous SGD: pack the gradient lists, sum them, move every
            worker by the sum and leave the sum in every gradient
  pack, unpack   between the lists and the flat copies
  broadcast one buffer into every copy

A case says which pass, on which layout, for how many workers, with binary32 or
bfloat16 gradients, and the group: one of the framework's own ("tiny",
"resnet50", "vgg16", "many_small") or a generic one of `numel` elements in
`tensors` tensors of log-uniformly spread sizes.  Lists are per-layer tensors
that start on 512-byte boundaries, as an allocator gives them, or ("views")
pieces of one dense buffer per worker, at any alignment.
"""

import functools
import math
import random

import numpy as np
import torch

import paper_1801_03855_amd as tc
from paper_1801_03855_amd import workloads

ETA = float(np.float32(0.05))
ALPHA = float(np.float32(0.05))
TAU = 64


def listed():
    def case(name, op, layout, K, grad, group, lists="own", numel=0, tensors=0, multiple=0):
        return {"name": name, "op": op, "layout": layout, "K": K, "grad": grad, "group": group, "lists": lists,
                "numel": numel, "tensors": tensors, "multiple": multiple}

    return [
        # A toy model's iteration: every call is a few microseconds, and what
        # counts is how fast calls follow each other.
        case("tiny_step", "step", "separate", 2, "f32", "tiny"),
        # A small model, a few hundred thousand parameters, four workers: one
        # call per iteration, too little work to fill the chip for long.
        case("small_pipeline", "pipeline", "tensor", 4, "f32", "generic", "own", 303_114, 65, 2),
        # A model of a million odd-sized parameters, eight workers: the elastic
        # step alone, on buffers that fit in the caches.
        case("medium_easgd", "easgd", "separate", 8, "f32", "generic", "own", 1_205_339, 120, 1),
        # The gradient average of synchronous data parallelism, four workers.
        case("resnet50_reduce", "reduce", "separate", 4, "f32", "resnet50"),
        # The benchmark's iteration: eight workers, four calls, tensor layout.
        case("resnet50_step", "step", "tensor", 8, "f32", "resnet50"),
        # The same iteration as one call.
        case("resnet50_pipeline", "pipeline", "tensor", 8, "f32", "resnet50"),
        # The elastic step for a program that keeps K separate flat buffers.
        case("resnet50_easgd", "easgd", "separate", 8, "f32", "resnet50"),
        # The iterations between two exchanges, with bfloat16 gradients.
        case("resnet50_period", "period", "separate", 8, "bf16", "resnet50"),
        # The largest model, gradient average and elastic step in one call.
        case("vgg16_fused", "fused", "separate", 4, "f32", "vgg16"),
        # Ten thousand small, mostly odd-sized tensors, sixteen workers,
        # bfloat16 gradients, in one call.
        case("many_small_pipeline", "pipeline", "tensor", 16, "bf16", "many_small"),
        # Synchronous SGD of five workers whose gradients are views of one
        # bucket per worker, at any alignment.
        case("ragged_pushpull", "pushpull", "separate", 5, "f32", "generic", "views", 9_000_011, 333, 1),
        # Asynchronous exchanges of a large set of workers.
        case("many_workers_async", "async", "tensor", 32, "f32", "generic", "own", 8_400_003, 200, 1),
    ]


# A pass costs no more than the largest listed one; at most 24 workers on
# separate buffers, which a pass returns one by one.
_MOST_ELEMENTS = 5.0e8  # of all workers together
_OPS = ("step", "pipeline", "reduce", "easgd", "fused", "period", "async", "pushpull", "pack", "unpack", "broadcast")


def draw(rng):
    op = rng.choice(_OPS)
    layout = "tensor" if op == "pipeline" else rng.choice(("separate", "tensor"))
    K = int(round(math.exp(rng.uniform(math.log(1.2), math.log(24 if layout == "separate" else 64)))))
    # the pushpull's broadcast sums come back in gradients of their own type
    grad = "f32" if op == "pushpull" else rng.choice(("f32", "f32", "bf16"))
    numel = int(math.exp(rng.uniform(math.log(7_000), math.log(min(1.4e8, _MOST_ELEMENTS / K)))))
    tensors = int(math.exp(rng.uniform(0.0, math.log(min(4_000, numel / 64)))))
    multiple = rng.choice((1, 1, 2, 16, 64))
    numel = max(numel // multiple, tensors) * multiple
    return {"op": op, "layout": layout, "K": K, "grad": grad, "group": "generic", "lists": rng.choice(("own", "own", "views")),
            "numel": numel, "tensors": tensors, "multiple": multiple}


# ------------------------------------------------------------------- inputs

@functools.lru_cache(maxsize=32)
def _generic_sizes(numel, tensors, multiple):
    """`tensors` sizes, multiples of `multiple`, log-uniform over a factor of
    1,000, that add up to numel (which is a multiple of `multiple`)."""
    u = np.random.default_rng(numel + 7 * tensors).random(tensors)
    w = np.exp(u * math.log(1000.0))
    units = numel // multiple
    cut = np.floor(np.concatenate([[0.0], np.cumsum(w) / w.sum()]) * units + 0.5).astype(np.int64)
    cut[-1] = units
    return tuple(int(v) * multiple for v in np.diff(cut))


def _sizes(case):
    if case["group"] != "generic":
        return workloads.group_sizes(case["group"])
    return list(_generic_sizes(case["numel"], case["tensors"], case["multiple"]))


def _starts(case, sizes, element):
    """Where each tensor of a list starts in its worker's storage, and the storage's length, in elements."""
    own = case["lists"] == "own"
    line = 512 // element
    at, starts = 0, []
    for s in sizes:
        starts.append(at)
        at += -(-s // line) * line if own else s
    return starts, at


def _rho(case):
    return float(np.float32(0.9 / (case["K"] * ETA)))


def _uses(case):
    """Which inputs the pass has."""
    return {"step": "gxc", "pipeline": "gxc", "reduce": "g", "easgd": "gxc", "fused": "gxc", "period": "gxc",
            "async": "xc", "pushpull": "gx", "pack": "g", "unpack": "g", "broadcast": "g"}[case["op"]]


def _inputs(case, seed, numel):
    """Flat values of every worker: gradients N(0, 0.01), workers N(0, 0.05)
    and a center that has drifted from their mean by N(0, 0.001)."""
    K = case["K"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    uses = _uses(case)
    gs, xs, xc = [], [], None
    if "g" in uses:
        for _ in range(1 if case["op"] == "broadcast" else K):
            g = torch.randn(numel, generator=gen, device="cuda").mul_(0.01)
            gs.append(g.to(torch.bfloat16) if case["grad"] == "bf16" else g)
    if "x" in uses:
        xs = [torch.randn(numel, generator=gen, device="cuda").mul_(0.05) for _ in range(K)]
    if "c" in uses:
        xc = torch.randn(numel, generator=gen, device="cuda").mul_(0.001)
        for x in xs:
            xc.add_(x, alpha=1.0 / K)
    order = list(range(K))
    random.Random(int(seed)).shuffle(order)
    return gs, xs, xc, order


def _interleaved(copies):
    """K flat copies as one tensor-layout buffer (element e of copy i at ((e // 4) * K + i) * 4 + e % 4)."""
    K, n = len(copies), copies[0].numel()
    slots = -(-n // 4)
    out = torch.zeros(slots, K, 4, dtype=copies[0].dtype, device=copies[0].device)
    for i, c in enumerate(copies):
        out[: n // 4, i] = c[: n // 4 * 4].view(-1, 4)
        if n % 4:
            out[-1, i, : n % 4] = c[n // 4 * 4:]
    return out.view(-1)


def _storage(case, sizes, copies, dtype=None, fill=True):
    """The per-layer tensors' storage of every worker, [K, length], with the copies' values in place."""
    dtype = dtype or copies[0].dtype
    starts, length = _starts(case, sizes, 2 if case["grad"] == "bf16" and dtype != torch.float32 else 4)
    out = torch.zeros(case["K"], length, dtype=dtype, device="cuda")
    if fill:
        where = _where(case, sizes, starts)
        for row, c in zip(out, copies):
            if where is None:
                row.copy_(c)
            else:
                row[where] = c.to(dtype)
    return out


def _where(case, sizes, starts):
    """The storage position of every flat element; None if they are the same."""
    if case["lists"] != "own":
        return None
    shift = np.asarray(starts, dtype=np.int64) - np.concatenate([[0], np.cumsum(sizes)[:-1]])
    n = int(sum(sizes))
    t = torch.repeat_interleave(torch.from_numpy(shift).cuda(), torch.tensor(sizes, device="cuda"), output_size=n)
    return t.add_(torch.arange(n, device="cuda"))


def _views(case, sizes, storage):
    """The storage's per-layer tensors, one list per worker."""
    starts, length = _starts(case, sizes, storage.element_size())
    cuts = []
    for s, a, b in zip(sizes, starts, starts[1:] + [length]):
        cuts += [s, b - a - s]
    return [list(row.split(cuts)[::2]) for row in storage]


# ------------------------------------------------------------- the interface

def prepare(case, seed):
    sizes = _sizes(case)
    group = tc.Group(sizes)
    n, K, op = group.numel, case["K"], case["op"]
    tensor = case["layout"] == "tensor"
    gdt = torch.bfloat16 if case["grad"] == "bf16" else torch.float32
    gs, xs, xc, order = _inputs(case, seed, n)
    s = {"case": case, "group": group, "K": K, "xc": xc, "order": order, "rho": _rho(case)}
    if xs:
        s["x"] = _interleaved(xs) if tensor else xs
    if op in ("step", "pipeline", "pushpull", "pack"):  # the gradients are in the workers' per-layer tensors
        s["grads"] = tc.TensorList(group, _views(case, sizes, _storage(case, sizes, gs)))
        s["g"] = (torch.zeros(tc.tensor_numel(group, K), dtype=gdt, device="cuda") if tensor
                  else [torch.zeros(n, dtype=gdt, device="cuda") for _ in range(K)])
    elif op == "broadcast":
        s["src"] = gs[0]
        s["g"] = (torch.zeros(tc.tensor_numel(group, K), dtype=gdt, device="cuda") if tensor
                  else [torch.zeros(n, dtype=gdt, device="cuda") for _ in range(K)])
    elif gs:
        s["g"] = _interleaved(gs) if tensor else gs
    if op in ("step", "pipeline", "unpack"):
        s["storage"] = _storage(case, sizes, gs, dtype=gdt if op == "unpack" else torch.float32, fill=False)
        s["params"] = tc.TensorList(group, _views(case, sizes, s["storage"]))
    if op in ("step", "pipeline", "reduce", "fused"):
        s["mean"] = torch.zeros(n, device="cuda")
    return s


def run(s):
    case, group, K = s["case"], s["group"], s["K"]
    op, tensor = case["op"], case["layout"] == "tensor"
    if op == "step" and tensor:
        tc.pack_tensor(s["grads"], s["g"])
        tc.reduce_tensor(group, K, s["g"], s["mean"], "avg")
        tc.easgd_step_tensor(group, K, s["x"], s["g"], s["xc"], ETA, s["rho"])
        tc.unpack_tensor(s["params"], s["x"])
    elif op == "step":
        tc.pack(s["grads"], s["g"])
        tc.reduce(group, s["g"], s["mean"], "avg")
        tc.easgd_step(group, s["x"], s["g"], s["xc"], ETA, s["rho"])
        tc.unpack(s["params"], s["x"])
    elif op == "pipeline":
        tc.easgd_pipeline_tensor(s["grads"], s["params"], s["g"], s["mean"], s["x"], s["xc"], ETA, s["rho"])
    elif op == "reduce" and tensor:
        tc.reduce_tensor(group, K, s["g"], s["mean"], "avg")
    elif op == "reduce":
        tc.reduce(group, s["g"], s["mean"], "avg")
    elif op == "easgd" and tensor:
        tc.easgd_step_tensor(group, K, s["x"], s["g"], s["xc"], ETA, s["rho"])
    elif op == "easgd":
        tc.easgd_step(group, s["x"], s["g"], s["xc"], ETA, s["rho"])
    elif op == "fused" and tensor:
        tc.reduce_easgd_step_tensor(group, K, s["x"], s["g"], s["xc"], s["mean"], ETA, s["rho"], "avg")
    elif op == "fused":
        tc.reduce_easgd_step(group, s["x"], s["g"], s["xc"], s["mean"], ETA, s["rho"], "avg")
    elif op == "period" and tensor:
        tc.easgd_period_step_tensor(group, K, s["x"], s["g"], s["xc"], ETA, s["rho"], 1, TAU)
    elif op == "period":
        tc.easgd_period_step(group, s["x"], s["g"], s["xc"], ETA, s["rho"], 1, TAU)
    elif op == "async" and tensor:
        tc.elastic_async_tensor(group, K, s["x"], s["xc"], s["order"], ALPHA)
    elif op == "async":
        tc.elastic_async(group, s["x"], s["xc"], s["order"], ALPHA)
    elif op == "pushpull" and tensor:
        tc.pack_tensor(s["grads"], s["g"])
        tc.sync_sgd_step_tensor(group, K, s["x"], s["g"], ETA, 1.0 / K, True)
    elif op == "pushpull":
        tc.pack(s["grads"], s["g"])
        tc.sync_sgd_step(group, s["x"], s["g"], ETA, 1.0 / K, True)
    elif op == "pack" and tensor:
        tc.pack_tensor(s["grads"], s["g"])
    elif op == "pack":
        tc.pack(s["grads"], s["g"])
    elif op == "unpack" and tensor:
        tc.unpack_tensor(s["params"], s["g"])
    elif op == "unpack":
        tc.unpack(s["params"], s["g"])
    elif op == "broadcast" and tensor:
        tc.broadcast_tensor(group, K, s["src"], s["g"])
    elif op == "broadcast":
        tc.broadcast(group, s["src"], s["g"])
    written = {"step": ("g", "mean", "x", "xc", "storage"), "pipeline": ("g", "mean", "x", "xc", "storage"),
               "reduce": ("mean",), "easgd": ("x", "xc"), "fused": ("mean", "x", "xc"), "period": ("x",),
               "async": ("x", "xc"), "pushpull": ("g", "x"), "pack": ("g",), "unpack": ("storage",), "broadcast": ("g",)}
    return {k: s[k] for k in written[op]}


def work(case):
    n, K = sum(_sizes(case)), case["K"]
    g = 2 if case["grad"] == "bf16" else 4
    # per element of the group: (bytes, operations)
    per = {"step": ((2 * g + 12) * K + 12, 7 * K + 3), "pipeline": ((2 * g + 12) * K + 12, 7 * K + 3),
           "reduce": (g * K + 4, K), "easgd": ((8 + g) * K + 8, 6 * K + 2), "fused": ((8 + g) * K + 12, 7 * K + 3),
           "period": ((8 + g) * K, 2 * K), "async": (8 * K + 8, 5 * K), "pushpull": ((2 * g + 8) * K, 3 * K),
           "pack": (2 * g * K, 0), "unpack": (2 * g * K, 0), "broadcast": (g + g * K, 0)}
    b, f = per[case["op"]]
    return {"bytes": b * n, "flops": f * n}


def tolerance(case):
    if case["op"] in ("pack", "unpack", "broadcast"):
        return "exact"
    # binary32 sums and updates, also from bfloat16 gradients
    return {"rel": 4e-7, "max": 4e-6}


def exact(case, seed):
    if case["op"] in ("pack", "unpack", "broadcast"):
        return None
    sizes = _sizes(case)
    n, K, op = sum(sizes), case["K"], case["op"]
    tensor = case["layout"] == "tensor"
    gs, xs, xc, order = _inputs(case, seed, n)
    eta, rho = ETA, _rho(case)
    out = {}
    if op in ("step", "pipeline", "reduce", "fused"):
        mean = torch.zeros(n, dtype=torch.float64, device="cuda")
        for g in gs:
            mean += g.double()
        out["mean"] = mean / K
    if op in ("step", "pipeline", "easgd", "fused"):
        c = xc.double()
        spread = torch.zeros_like(c)
        new = []
        for x, g in zip(xs, gs):
            d = x.double() - c
            spread += d
            new.append(x.double() - eta * (g.double() + rho * d))
        out["x"], out["xc"] = new, c + eta * rho * spread
    elif op == "period":
        out["x"] = [x.double() - eta * g.double() for x, g in zip(xs, gs)]
    elif op == "async":
        c, new = xc.double(), [x.double() for x in xs]
        for w in order:
            d = new[w] - c
            c = c + ALPHA * d
            new[w] = new[w] - ALPHA * d
        out["x"], out["xc"] = new, c
    elif op == "pushpull":
        total = torch.zeros(n, dtype=torch.float64, device="cuda")
        for g in gs:
            total += g.double()
        out["x"] = [x.double() - eta / K * total for x in xs]
        out["g"] = [total] * K
    if op in ("step", "pipeline"):
        out["storage"] = _storage(case, sizes, out["x"], dtype=torch.float32, fill=False).double()
        starts, _ = _starts(case, sizes, 4)
        where = _where(case, sizes, starts)
        for row, x in zip(out["storage"], out["x"]):
            row[where if where is not None else slice(None)] = x
        out["g"] = None  # the gradients' own bits
    if tensor:
        out.update({k: _interleaved(out[k]) for k in ("x", "g") if isinstance(out.get(k), list)})
    return out
