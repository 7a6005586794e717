"""The work that performance is measured on: what users of the library have it do, over the sizes they do it at.

listed() names the standing cases, draw(rng) gives another case of the same ranges, prepare(case, seed) makes what
a program has in hand before the call, run(state) is one pass through the public entry points, work(case) says
what that pass cannot do without and tolerance(case) how far two correct results may lie apart.

Kinds of case:
  hops    the hop stack [X, A^X, ..] in device memory, on a plan that is kept (one plan, many feature matrices);
  filter  a constant polynomial filter sum_k c_k A^^k X without the stack;
  once    the whole precompute of a graph seen for the first time: plan its edge list, run the hops, drop the plan;
  plan    the edge list alone turned into a plan, on the host's threads or on the GPU;
  stream  the hop stack of operands that live in pinned host memory;
  model   the forward pass of an LC-version model over a mini-batch, or over all rows, of a hop stack.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import gp_synth
import paper_2207_12000_amd as gp

AGG = {"sym": gp.GP_AGG_SYM, "mean": gp.GP_AGG_MEAN, "sum": gp.GP_AGG_SUM}
TORCH_TYPE = {"f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "bf16": 2}
COMMUNITIES = 50          # of the community graphs; 90 % of the draws fall inside one
HIDDEN, CLASSES = 256, 40  # widths of the model's hidden layers and of its output


def listed():
    return [
        # the smallest graphs (a citation network of a few thousand papers): launches and latency are all there is
        dict(name="tiny_sym", kind="hops", graph="uniform", n=10_000, pairs=100_000, d=128, dtype="f32", agg="sym",
             loops=True, K=2, budget=52_500, plan="host"),
        # a small graph of odd sizes: rows of 47 columns start on no 16-byte boundary, some rows have no source
        dict(name="odd_mean", kind="hops", graph="powerlaw", n=37_123, pairs=411_007, gamma=2.1, hub=900, d=47,
             dtype="f32", agg="mean", loops=False, K=4, budget=1 << 20, plan="host"),
        # an arxiv-sized citation graph, the precompute of a simplified-GCN / LC model
        dict(name="citation_sym", kind="hops", graph="powerlaw", n=169_343, pairs=1_166_243, gamma=2.1, hub=1000,
             d=128, dtype="f32", agg="sym", loops=True, K=3, budget=1 << 20, plan="host"),
        # the same kind of graph stored in bf16, three times as large
        dict(name="citation_sym_bf16", kind="hops", graph="powerlaw", n=507_001, pairs=4_900_000, gamma=2.1, hub=3000,
             d=128, dtype="bf16", agg="sym", loops=True, K=3, budget=1 << 22, plan="device"),
        # a products-sized co-purchase graph: heavy hubs, 400-byte rows, nothing fits a cache
        dict(name="powerlaw_mean", kind="hops", graph="powerlaw", n=2_450_000, pairs=61_900_000, gamma=2.0, hub=10_000,
             d=100, dtype="f32", agg="mean", loops=False, K=3, budget=8_000_000, plan="device"),
        # a Reddit-sized community graph: mean degree near 500 and 602 columns, the largest in-memory precompute
        dict(name="community_sum", kind="hops", graph="community", n=233_000, pairs=57_000_000, d=602, dtype="f32",
             agg="sum", loops=True, K=2, budget=8_000_000, plan="device"),
        # ten steps of Personalized PageRank diffusion over 64 columns
        dict(name="filter_ppr", kind="filter", graph="powerlaw", n=169_343, pairs=1_166_243, gamma=2.1, hub=1000, d=64,
             dtype="f32", agg="sym", loops=True, K=10, budget=1 << 20, plan="host"),
        # a graph's only precompute, from its edge list to the stack
        dict(name="once_sym", kind="once", graph="powerlaw", n=490_000, pairs=6_000_000, gamma=2.1, hub=4000, d=100,
             dtype="f32", agg="sym", loops=True, K=3, budget=8_000_000, plan="device"),
        # planning on the host's threads, as a program without a free GPU does
        dict(name="plan_host", kind="plan", graph="powerlaw", n=490_000, pairs=6_000_000, gamma=2.1, hub=4000,
             loops=True, budget=1 << 22, plan="host"),
        # a stack that stays in host memory, streamed through the GPU
        dict(name="stream_sym_bf16", kind="stream", graph="powerlaw", n=1_110_600, pairs=16_157_000, gamma=2.1, hub=10_000,
             d=128, dtype="bf16", agg="sym", loops=True, K=3, budget=1 << 22, plan="device"),
        # one mini-batch of inference: four hops, four layers, then the softmax
        dict(name="model_batch", kind="model", n=169_343, d=128, dtype="f32", K=3, layers=4, batch=4096, form="sum"),
        # all rows at once through branches of growing depth, side by side, from a bf16 stack of odd width
        dict(name="model_all_bf16", kind="model", n=169_343, d=100, dtype="bf16", K=3, layers=3, batch=0, form="concat"),
    ]


def draw(rng):
    """One more case of the ranges above.  Sizes are spread over their logarithms."""
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["hops", "hops", "hops", "hops", "filter", "once", "plan", "stream", "model", "model"])
    c = dict(kind=kind)
    if kind == "model":
        c.update(n=size(20_000, 200_000), d=size(32, 320), dtype=rng.choice(["f32", "bf16"]), K=rng.randint(1, 4),
                 layers=rng.randint(2, 4), form=rng.choice(["sum", "sum", "concat", "max"]),
                 batch=rng.choice([0, size(512, 16_384)]))
        return c
    graph = rng.choice(["uniform", "powerlaw", "powerlaw", "community"]) if kind == "hops" else "powerlaw"
    c["graph"] = graph
    if graph == "community":
        c["n"] = COMMUNITIES * size(400, 4_660)
        c["pairs"] = int(c["n"] * rng.uniform(20, min(250, c["n"] / COMMUNITIES / 8)))
    else:
        c["n"] = size(3_000, 1_500_000)
        c["pairs"] = int(c["n"] * math.exp(rng.uniform(math.log(4), math.log(25))))
        if graph == "powerlaw":
            c["gamma"], c["hub"] = round(rng.uniform(2.0, 2.4), 2), int(min(c["n"] / 8, rng.uniform(200, 10_000)))
    if kind in ("once", "plan", "stream"):
        c["n"] = min(c["n"], 1_000_000)
        c["pairs"] = min(c["pairs"], 16_000_000)
    c["loops"] = rng.random() < 0.6
    c["budget"] = rng.choice([1 << 20, 1 << 22, 8_000_000])
    c["plan"] = rng.choice(["host", "device"]) if kind in ("once", "plan") else "host" if c["pairs"] < 4_000_000 else "device"
    if kind == "plan":
        return c
    c["dtype"] = "bf16" if kind == "stream" else rng.choice(["f32", "f32", "bf16"])
    c["d"] = rng.choice([64, 100, 128, 256, size(16, 640), size(16, 640)])
    if kind == "stream":
        c["d"] = rng.choice([64, 128, 256])
    c["agg"] = rng.choice(["sym", "sym", "mean", "sum"])
    c["K"] = rng.randint(2, 10) if kind == "filter" else rng.randint(1, 4)
    # no more work than the largest listed case of the kind
    c["d"] = max(16, min(c["d"], int({"hops": 2e10, "filter": 3e9, "once": 3e9, "stream": 1.2e10}[kind] / (nonzeros(c) * c["K"]))))
    if kind == "stream":
        c["d"] -= c["d"] % 8
    return c


def nonzeros(c):
    """Stored non-zeros: both directions of every distinct pair, and the diagonal."""
    return 2 * c["pairs"] + (c["n"] if c.get("loops", True) else 0)


# ---- inputs ----------------------------------------------------------------------------------------

def _draw_pairs(c, m, gen):
    """m unordered pairs in keys lo * n + hi, repeats and all."""
    n, dev = c["n"], "cuda"

    def ids(bound):
        return torch.randint(bound, (m,), generator=gen, device=dev)

    if c["graph"] == "uniform":
        u, v = ids(n), ids(n)
    elif c["graph"] == "community":
        s = n // COMMUNITIES
        u, inside = ids(n), torch.rand(m, generator=gen, device=dev) < 0.9
        shift = (1 + ids(COMMUNITIES - 1)).masked_fill_(inside, 0)
        v = (u // s + shift) % COMMUNITIES * s + ids(s)
    else:  # expected degrees fall with a power of the rank
        a = 1.0 / (c["gamma"] - 1.0)
        i0 = gp_synth.chung_lu_offset(n, 2 * c["pairs"], c["gamma"], float(c["hub"]))

        def ranks():
            r = torch.rand(m, generator=gen, device=dev, dtype=torch.float64)
            if abs(a - 1.0) < 1e-9:
                x = i0 * torch.exp(r * math.log((n + i0) / i0)) - i0
            else:
                lo, hi = i0 ** (1.0 - a), (n + i0) ** (1.0 - a)
                x = (lo + r * (hi - lo)) ** (1.0 / (1.0 - a)) - i0
            return x.long().clamp_(0, n - 1)

        u, v = ranks(), ranks()
    keep = u != v
    return (torch.minimum(u, v) * n + torch.maximum(u, v))[keep]


def _edges(c, gen):
    """The case's edge list on the host, drawn on the GPU: `pairs` distinct pairs in no order, then every twentieth
    of them once more the other way round.  Ids carry no locality."""
    n, m = c["n"], c["pairs"]
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < m:
        keys = torch.unique(torch.cat([keys, _draw_pairs(c, int((m - keys.numel()) * 1.15) + 64, gen)]))
    keys = keys[torch.randperm(keys.numel(), generator=gen, device="cuda")[:m]]
    perm = torch.randperm(n, generator=gen, device="cuda").to(torch.int32)
    u, v = perm[keys // n], perm[keys % n]
    return torch.cat([u, v[::20]]).cpu().numpy(), torch.cat([v, u[::20]]).cpu().numpy()


def _flags(c):
    return (gp.GP_SYMMETRISE | (gp.GP_ADD_SELF_LOOPS if c.get("loops", True) else 0) |
            (gp.GP_PLAN_ON_DEVICE if c.get("plan") == "device" else 0))


def _plan(c, src, dst):
    return gp.gp_plan_blocks(src, dst, c["n"], c.get("budget", 1 << 20), _flags(c))


def prepare(case, seed):
    c = dict(case)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if c["kind"] == "model":
        return _prepare_model(c, gen)
    src, dst = _edges(c, gen)
    if c["kind"] == "plan":
        return dict(c=c, src=src, dst=dst)
    X = torch.randn(c["n"], c["d"], generator=gen, device="cuda").to(TORCH_TYPE[c["dtype"]])
    if c["kind"] == "once":
        return dict(c=c, src=src, dst=dst, X=X)
    plan = _plan(c, src, dst)
    if c["kind"] == "hops":
        return dict(c=c, plan=plan, X=X)
    if c["kind"] == "filter":
        alpha = 0.1
        coeff = [alpha * (1 - alpha) ** k for k in range(c["K"])] + [(1 - alpha) ** c["K"]]
        return dict(c=c, plan=plan, X=X, coeff=coeff)
    # streamed: slab 0 of the stack holds X already
    stack = torch.empty(c["K"] + 1, c["n"], c["d"], dtype=X.dtype, pin_memory=True)
    stack[0].copy_(X)
    return dict(c=c, plan=plan, stack=stack)


def _prepare_model(c, gen):
    """A stack (features halve with every hop, as averages over neighbours do), a batch of rows, weights, and one
    coefficient per hop."""
    stack = torch.empty(c["K"] + 1, c["n"], c["d"], dtype=TORCH_TYPE[c["dtype"]], device="cuda")
    for k in range(c["K"] + 1):
        stack[k] = torch.randn(c["n"], c["d"], generator=gen, device="cuda") * 0.5 ** k
    batch = torch.randperm(c["n"], generator=gen, device="cuda")[:c["batch"]].to(torch.int32) if c["batch"] else None
    widths = _widths(c)
    weights = [torch.randn(i, o, generator=gen, device="cuda") / math.sqrt(i) for i, o in zip([c["d"]] + widths, widths)]
    gamma = [0.1 * 0.9 ** k for k in range(c["K"])] + [0.9 ** c["K"]]
    return dict(c=c, stack=stack, batch=batch, weights=weights, gamma=gamma, depth=_depth(c))


def _widths(c):
    return [HIDDEN] * (c["layers"] - 1) + [CLASSES if c["form"] == "sum" else HIDDEN]


def _depth(c):
    """Layers every hop's branch applies: all of them, or as many as its hop count (hop 0 left out)."""
    if c["form"] == "sum":
        return None
    return [min(k, c["layers"]) for k in range(c["K"] + 1)]


# ---- one pass --------------------------------------------------------------------------------------

class _Held:
    """An array of a plan that keeps the plan alive (np.asarray of it has this object as its base)."""

    def __init__(self, plan, view):
        self.plan, self.__array_interface__ = plan, view.__array_interface__


def run(state):
    c = state["c"]
    if c["kind"] == "hops":
        return gp.propagate_tensors(state["plan"], state["X"], AGG[c["agg"]], c["K"])
    if c["kind"] == "filter":
        X = state["X"]
        out = torch.empty_like(X)
        gp.gp_propagate_combine(state["plan"], X.data_ptr(), X.stride(0), c["d"], gp.GP_F32 if c["dtype"] == "f32" else gp.GP_BF16,
                                AGG[c["agg"]], c["K"], state["coeff"], out.data_ptr(), out.stride(0),
                                torch.cuda.current_stream().cuda_stream)
        return out
    if c["kind"] == "once":
        with _plan(c, state["src"], state["dst"]) as plan:
            return gp.propagate_tensors(plan, state["X"], AGG[c["agg"]], c["K"])
    if c["kind"] == "plan":
        plan = _plan(c, state["src"], state["dst"])
        names = ("rowptr", "col", "deg", "dinv_sqrt", "dinv", "block_off", "block_row_lo", "block_row_hi")
        return {k: np.asarray(_Held(plan, getattr(plan, k))) for k in names}
    if c["kind"] == "stream":
        return gp.propagate_tensors(state["plan"], state["stack"][0], AGG[c["agg"]], c["K"], out=state["stack"])
    comb = {"sum": gp.GP_COMB_SUM, "concat": gp.GP_COMB_CONCAT, "max": gp.GP_COMB_MAX}[c["form"]]
    H = gp.lc_forward_tensors(state["stack"], state["batch"], state["gamma"], state["weights"], depth=state["depth"], comb=comb)
    if c["form"] == "sum":
        gp.gp_lc_softmax(H.data_ptr(), H.shape[0], H.shape[1], H.stride(0), torch.cuda.current_stream().cuda_stream)
    return H


# ---- what a pass cannot do without, and how close two results are ----------------------------------

def _listed_pairs(c):
    return c["pairs"] + (c["pairs"] + 19) // 20


def work(case):
    c = dict(case)
    n = c["n"]
    if c["kind"] == "model":
        rows = c["batch"] or n
        widths, depth = _widths(c), _depth(c) or [c["layers"]] * (c["K"] + 1)
        shapes = list(zip([c["d"]] + widths, widths))
        ends = [widths[k - 1] for k in depth if k]
        out = sum(ends) if c["form"] == "concat" else ends[0]
        return {"bytes": rows * (len(ends) * c["d"] * BYTES[c["dtype"]] + 4 * out) + 4 * sum(i * o for i, o in shapes),
                "flops": 2 * rows * sum(sum(i * o for i, o in shapes[:k]) for k in depth)}
    nnz = nonzeros(c)
    lists = 4 * nnz + 8 * (n + 1)
    if c["kind"] == "plan":
        return {"bytes": 8 * _listed_pairs(c) + lists + 12 * n, "flops": 0}
    slab = n * c["d"] * BYTES[c["dtype"]]
    stack = 2 if c["kind"] == "filter" else c["K"] + (1 if c["kind"] == "stream" else 2)  # X read, what is returned written
    return {"bytes": stack * slab + lists + (8 * _listed_pairs(c) if c["kind"] == "once" else 0), "flops": 2 * nnz * c["d"] * c["K"]}


def tolerance(case):
    """About four times the most that results were seen to differ by with the same sums taken in another order
    (segments of another length, hot rows gathered apart or not), or, for the model, from a computation in fp64."""
    if case["kind"] == "plan":
        return "exact"
    if case["kind"] == "model":
        return {"rel": 1.2e-6, "max": 1.2e-5}
    if case["dtype"] == "bf16":  # every hop is rounded to bf16: a sum taken in another order now and then rounds the other way
        return {"rel": 4e-5, "max": 3e-2}
    return {"rel": 5e-7, "max": 2e-5}
