"""Performance cases: what a user of the library has it do, through its public entry points.

A case is one mini-batch (or one group of mini-batches) of split-parallel GNN training or inference on
a seeded power-law graph: sampling and splitting, loading of the input features, and the model.  Sizes
follow the repository's own workloads (`workloads/synth.py`: tiny, medium, large, skewed, sweep; the two
largest graphs with fewer vertices, so that their inputs are made in a second); the others are generic.
Keys of a case:

  kind      train     sampling, loading, GraphSAGE forward, loss and backward
            infer     sampling, loading, GraphSAGE forward (serving, evaluation)
            gat       sampling, loading, GAT forward, loss and backward
            group     the sampling and loading of `group` mini-batches in one set of launches
            presample sampling and the counts of the offline partitioning weights
            cached    sampling and loading through the feature cache, misses from pinned host memory
  vertices, degree   the graph: R-MAT, degree = directed edges drawn per vertex before duplicates go
  skew      probability of the heaviest R-MAT quadrant (0.57; 0.6 with the other three alike is the skewed graph)
  symmetric, permuted, wide   both directions of an edge stored; ids shuffled; 64-bit row pointers
  splits, map        logical splits and the partition map ("random" or "range")
  batch, fanouts     targets; fanouts[l] expands level l + 1 into level l
  dims, dtype        layer widths (dims[0] input features, dims[-1] classes); "f32" or "bf16"
  heads     GAT: attention heads of the hidden layers
  calls     train: "step" = the one-call step, "separate" = forward, loss, backward as three calls
  cached    share of every split's vertices whose features the cache holds
"""
import math
import random

import torch

from paper_2303_13775_amd import (GSPLIT_BF16, GSPLIT_F32, Context, GatParams, SageParams, gsplit_gather_features_multi,
                                  gsplit_sample_split_multi)

SAMPLE_SEED = 0xC0FFEE

_BASE = {"kind": "train", "vertices": 2_400_000, "degree": 54, "skew": 0.57, "symmetric": True, "permuted": True,
         "wide": False, "splits": 4, "map": "range", "batch": 1024, "fanouts": "15,10,5", "dims": "100,256,256,47",
         "dtype": "f32", "heads": 4, "group": 1, "calls": "step", "cached": 0.0}


def _case(name, **over):
    return dict(_BASE, name=name, **over)


def listed():
    return [
        # serving: the classes of a handful of vertices on request; launches and latency are all of it
        _case("serve_33", kind="infer", batch=33),
        # the tiny workload's training step
        _case("tiny_train", vertices=1 << 14, degree=32, permuted=False, map="random", fanouts="10,5", dims="64,64,16"),
        # nothing a multiple of anything: graph, batch, widths, splits, and the model as three calls
        _case("ragged_train", vertices=99_991, degree=19, splits=3, map="random", batch=777, fanouts="7,3,5",
              dims="50,130,70,19", calls="separate"),
        # the benchmark workload, float32 and bf16
        _case("medium_train"),
        _case("medium_train_bf16", dtype="bf16"),
        # the second model on it, heads 4-4-1
        _case("medium_gat", kind="gat"),
        # the sampling stream of an overlapped trainer: eight mini-batches sampled and loaded ahead
        _case("medium_group", kind="group", group=8),
        # one iteration of the offline pre-sampling stage (a single split, edge positions recorded)
        _case("medium_presample", kind="presample", splits=1),
        # features in host memory, the hottest quarter of them cached
        _case("medium_cached", kind="cached", vertices=400_000, cached=0.25),
        # the large workload: one direction of every edge, 64-bit row pointers, 172 classes
        _case("large_train", vertices=1 << 24, degree=15, symmetric=False, wide=True, batch=4096, dims="128,256,256,172"),
        # hub vertices, ids not shuffled, wide fanouts
        _case("skewed_train", vertices=6_500_000, degree=56, skew=0.6, permuted=False, wide=True, batch=4096,
              fanouts="20,20,20", dims="128,256,256,64"),
        # the split sweep: four layers, eight splits, bf16
        _case("sweep_train_bf16", vertices=1 << 24, degree=15, symmetric=False, wide=True, splits=8, batch=8192,
              fanouts="10,10,10,10", dims="128,256,256,256,172", dtype="bf16"),
    ]


def draw(rng: random.Random):
    """One more case of the ranges the listed ones span."""
    def log_uniform(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choices(["train", "infer", "gat", "group", "presample", "cached"], [10, 3, 3, 2, 1, 1])[0]
    c = dict(_BASE, kind=kind)
    c["vertices"] = log_uniform(1 << 14, 400_000 if kind == "cached" else 1 << 24)
    c["degree"] = min(rng.randint(10, 56), max(10, 300_000_000 // c["vertices"]))
    if rng.random() < 0.25:
        c["skew"], c["permuted"] = 0.6, False
    c["symmetric"] = rng.random() < 0.7
    c["wide"] = rng.random() < 0.4
    c["splits"] = 1 if kind == "presample" else rng.choice([1, 2, 3, 4, 4, 8])
    c["map"] = rng.choice(["random", "range"])
    c["batch"] = min(log_uniform(16, 8192), c["vertices"] // 8)
    layers = rng.choice([2, 3, 3, 3, 4])
    c["fanouts"] = ",".join(str(rng.choice([3, 5, 7, 10, 10, 15] + ([20, 25] if layers < 4 else []))) for _ in range(layers))
    hidden = rng.choice([64, 128, 256, 256, 4 * rng.randint(8, 64)])
    c["dims"] = ",".join(str(x) for x in [4 * rng.randint(8, 64)] + [hidden] * (layers - 1) + [rng.randint(5, 180)])
    if kind in ("train", "infer"):
        c["dtype"] = rng.choice(["f32", "f32", "bf16"])
        c["calls"] = rng.choice(["step", "step", "separate"])
        if c["dtype"] == "f32" and rng.random() < 0.3:      # widths that are not multiples of 4
            c["dims"] = ",".join(str(x) for x in [rng.randint(30, 250)] + [rng.randint(30, 250) for _ in range(layers - 1)]
                                 + [rng.randint(5, 180)])
    if kind == "gat":
        c["heads"] = rng.choice([1, 2, 4, 4])
    if kind == "group":
        c["group"] = rng.choice([2, 4, 8])
    if kind == "cached":
        c["cached"] = round(rng.uniform(0.1, 0.9), 3)
    # a drawn case costs no more than the largest listed one, and its buffers (sized by the bound on the
    # rows of every level) fit the card several times over
    most = max(_cost(x) for x in listed())
    while c["batch"] > 16 and (_cost(c) > 0.6 * most or _memory(c) > 30e9):
        c["batch"] = max(16, int(c["batch"] * 0.7))
    return c


def _ints(text):
    return [int(x) for x in text.split(",")]


def _memory(c):
    """Bytes of a state's buffers, which are sized by the no-duplicates bound on the rows of every level."""
    dims, fan, rows, total = _ints(c["dims"]), _ints(c["fanouts"]), c["batch"], 0
    el = 2 if c["dtype"] == "bf16" else 4
    for l in range(len(fan) - 1, -1, -1):
        total += rows * (1 + fan[l]) * 60 + (0 if c["kind"] in ("group", "cached", "presample") else
                                             rows * 4 * (dims[l + 1] + 2 * max(dims[l], c["heads"] * dims[l] // 2)))
        rows = min(c["vertices"], rows * (1 + fan[l]))
    if c["kind"] == "gat" and (dims[1] // c["heads"]) % 4:
        total += rows * 8 * (dims[1] + 2 * c["heads"])
    return c["group"] * (total + rows * dims[0] * el) + c["vertices"] * (4 * c["degree"] + dims[0] * el)


def _graph(c, gen, dev):
    """R-MAT graph: CSR without duplicates or self loops (the edge array has room for all pairs drawn, so
    that its size does not depend on how many were duplicates)."""
    n, a = c["vertices"], c["skew"]
    b = 0.19 if a == 0.57 else 0.15
    pairs = n * c["degree"] // (2 if c["symmetric"] else 1)
    perm = torch.randperm(n, generator=gen, device=dev) if c["permuted"] else None
    keys = []
    for done in range(0, pairs, 1 << 26):
        m = min(1 << 26, pairs - done)
        src = torch.zeros(m, dtype=torch.int32, device=dev)
        dst = torch.zeros(m, dtype=torch.int32, device=dev)
        for _ in range((n - 1).bit_length()):
            u = torch.rand(m, generator=gen, device=dev)
            s = u >= a + b
            src = src * 2 + s
            dst = dst * 2 + torch.where(s, u >= a + 2 * b, u >= a)
        keep = (src != dst) & (src < n) & (dst < n)
        src, dst = src[keep].long(), dst[keep].long()
        if perm is not None:
            src, dst = perm[src], perm[dst]
        keys.append(src * n + dst)
        if c["symmetric"]:
            keys.append(dst * n + src)
    keys = torch.unique(torch.cat(keys))
    indptr = torch.searchsorted(keys, torch.arange(n + 1, device=dev) * n)
    indices = torch.zeros(pairs * (2 if c["symmetric"] else 1), dtype=torch.int32, device=dev)
    indices[:keys.numel()] = keys % n
    return indptr if c["wide"] else indptr.to(torch.int32), indices


def _uniform(shape, limit, gen, dev):
    return (torch.rand(shape, generator=gen, device=dev) * 2 - 1) * limit


class _State:
    pass


def prepare(case, seed):
    c, dev = dict(_BASE, **case), torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed) * 1_000_003 + 17)
    s = _State()
    s.kind, s.calls = c["kind"], c["calls"]
    n, S, fan, dims, batch = c["vertices"], c["splits"], _ints(c["fanouts"]), _ints(c["dims"]), c["batch"]
    L = len(fan)
    s.indptr, s.indices = _graph(c, gen, dev)
    if c["map"] == "random":
        s.pmap = torch.randint(0, S, (n,), generator=gen, device=dev).to(torch.uint8)
    else:
        s.pmap = (torch.arange(n, device=dev) * S // n).to(torch.uint8)
    draw_ids = lambda: torch.randperm(n, generator=gen, device=dev)[:batch].to(torch.int32).contiguous()  # noqa: E731
    context = lambda: Context(s.indptr, s.indices, s.pmap, S, fan, batch, keep_edge_ids=s.kind == "presample",  # noqa: E731
                              gat_index=s.kind == "gat")
    s.ctx, s.targets, s.it = context(), draw_ids(), int(seed) & 0xFFFF
    if s.kind == "presample":
        s.vertex_count = torch.zeros(n, dtype=torch.int32, device=dev)
        s.edge_count = torch.zeros(s.indices.numel(), dtype=torch.int32, device=dev)
        return s
    store = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    feat = torch.empty((n, dims[0]), dtype=store, device=dev)
    for r in range(0, n, 1 << 22):
        feat[r:r + (1 << 22)] = torch.randn((min(n, r + (1 << 22)) - r, dims[0]), generator=gen, device=dev)
    if s.kind in ("group", "cached"):
        s.ctxs = [s.ctx] + [context() for _ in range(c["group"] - 1)]
        s.all_targets = [s.targets] + [draw_ids() for _ in range(c["group"] - 1)]
        s.its = [s.it + k for k in range(c["group"])]
        s.x0s = [torch.zeros((x.gsplit_max_rows(0), dims[0]), dtype=store, device=dev) for x in s.ctxs]
        s.feat = feat
        if s.kind == "cached":
            s.feat = torch.empty(feat.shape, dtype=store, pin_memory=True)
            s.feat.copy_(feat)
            # the hottest vertices of every split: many in-edges, many samples
            heat = torch.zeros(n, dtype=torch.int64, device=dev)
            live = s.indices[:int(s.indptr[-1])].long()
            heat.index_add_(0, live, torch.ones_like(live))
            ids, counts = [], []
            for k in range(S):
                own = torch.nonzero(s.pmap == k).flatten()
                own = own[torch.sort(heat[own], descending=True, stable=True).indices[:int(own.numel() * c["cached"])]]
                ids.append(own.to(torch.int32))
                counts.append(own.numel())
            s.ctx.gsplit_cache_build(s.feat, torch.cat(ids).contiguous(), counts)
        return s
    s.feat = feat
    s.x0 = torch.zeros((s.ctx.gsplit_max_rows(0), dims[0]), dtype=store, device=dev)
    s.labels = torch.randint(0, dims[-1], (n,), generator=gen, device=dev)
    s.logits = torch.empty((batch, dims[-1]), device=dev)
    s.grad_logits, s.row_loss = torch.empty_like(s.logits), torch.empty(batch, device=dev)
    if s.kind == "gat":
        heads = [c["heads"]] * (L - 1) + [1]
        per_head = [dims[l + 1] // heads[l] for l in range(L)]
        weights = [[], [], [], []]
        for l in range(L):
            width = heads[l] * per_head[l]
            weights[0].append(_uniform((dims[l], width), math.sqrt(6 / (dims[l] + width)), gen, dev))
            for k in (1, 2):
                weights[k].append(_uniform((width,), math.sqrt(6 / (per_head[l] + 1)), gen, dev))
            weights[3].append(_uniform((dims[l + 1],), 0.1, gen, dev))
        s.params = GatParams(dims, heads, *weights)
    else:
        weights = [[], [], []]
        for l in range(L):
            for k in (0, 1):
                weights[k].append(_uniform((dims[l], dims[l + 1]), math.sqrt(6 / (dims[l] + dims[l + 1])), gen, dev))
            weights[2].append(_uniform((dims[l + 1],), 0.1, gen, dev))
        s.params = SageParams(dims, *weights, dtype=GSPLIT_BF16 if store == torch.bfloat16 else GSPLIT_F32)
    s.weights = weights
    s.grads = [[torch.empty_like(t) for t in part] for part in weights]
    return s


def run(s):
    if s.kind == "group":
        gsplit_sample_split_multi(s.ctxs, s.all_targets, SAMPLE_SEED, s.its)
        gsplit_gather_features_multi(s.ctxs, s.feat, s.x0s)
        return s.x0s
    s.ctx.gsplit_sample_split(s.targets, SAMPLE_SEED, s.it)
    if s.kind == "presample":
        s.ctx.gsplit_presample_accumulate(s.vertex_count, s.edge_count)
        return s.vertex_count, s.edge_count
    if s.kind == "cached":
        s.ctx.gsplit_gather_features_cached(s.x0s[0])
        return s.x0s
    s.ctx.gsplit_gather_features(s.feat, s.x0)
    if s.kind == "infer":
        s.ctx.gsplit_sage_fwd(s.params, s.x0, s.logits)
        return {"rows": s.x0, "logits": s.logits}
    if s.kind == "gat":
        s.ctx.gsplit_gat_fwd(s.params, s.x0, s.logits)
        s.ctx.gsplit_softmax_xent(s.logits, s.labels, s.grad_logits, s.row_loss)
        s.ctx.gsplit_gat_bwd(s.params, s.x0, s.grad_logits, *s.grads)
    elif s.calls == "step":
        s.ctx.gsplit_sage_step(s.params, s.x0, s.labels, s.logits, *s.grads, row_loss=s.row_loss)
    else:
        s.ctx.gsplit_sage_fwd(s.params, s.x0, s.logits)
        s.ctx.gsplit_softmax_xent(s.logits, s.labels, s.grad_logits, s.row_loss)
        s.ctx.gsplit_sage_bwd(s.params, s.grad_logits, *s.grads)
    return {"rows": s.x0, "logits": s.logits, "loss": s.row_loss, "grads": s.grads}


def _levels(c):
    """Expected rows of every level and sampled edges of every layer.  A vertex whose id has k one bits
    draws an R-MAT endpoint with probability p_k, so levels are counted by k."""
    n, a = c["vertices"], c["skew"]
    b = 0.19 if a == 0.57 else 0.15
    bits = (n - 1).bit_length()
    count = [n * math.comb(bits, k) / 2 ** bits for k in range(bits + 1)]
    p = [(a + b) ** (bits - k) * (1 - a - b) ** k for k in range(bits + 1)]
    total = sum(x * y for x, y in zip(count, p))
    p = [x / total for x in p]
    degree = [n * c["degree"] * x for x in p]
    now = [c["batch"] * x / n for x in count]
    rows, edges = [sum(now)], []
    for f in reversed(_ints(c["fanouts"])):
        m = sum(x * f * (1 - math.exp(-d / f)) for x, d in zip(now, degree))
        edges.append(m)
        now = [x + (k - x) * (1 - math.exp(-m * q)) if k > 0 else 0.0 for x, k, q in zip(now, count, p)]
        rows.append(sum(now))
    return rows[::-1], edges[::-1]


def work(case):
    """Bytes and operations one pass cannot do without: rows of the graph, the features and the weights
    read once, the batch's index arrays, the loaded rows, logits and gradients written once; the products
    of the model with the expected number of rows of every level."""
    c = dict(_BASE, **case)
    dims, L = _ints(c["dims"]), len(_ints(c["fanouts"]))
    rows, edges = _levels(c)
    ptr, el = (16 if c["wide"] else 8), (2 if c["dtype"] == "bf16" else 4)
    # per destination: row pointers, count, block offset; per edge: neighbour id read, sampled id and
    # relabelled source written; per row of the new level: id, owner, mixed frontier, shuffle index
    total = 4.0 * c["batch"]
    for l in range(L):
        total += rows[l + 1] * (ptr + 8) + edges[l] * 12 + rows[l] * 13
    if c["kind"] == "presample":
        # two counters, read and written, per vertex above the input layer and per edge
        return {"bytes": total + 8 * sum(rows[1:]) + 8 * sum(edges), "flops": 0}
    total += rows[0] * (4 + 2 * dims[0] * el)
    if c["kind"] in ("group", "cached"):
        return {"bytes": c["group"] * total, "flops": 0}
    back = c["kind"] != "infer"
    flops, params = 0.0, 0
    for l in range(L):
        if c["kind"] == "gat":
            width = dims[l + 1]
            params += dims[l] * width + 3 * width
            products = 2 * rows[l + 1] * dims[l] * width + 4 * (rows[l + 1] + edges[l]) * max(dims[l], width)
        else:
            params += 2 * dims[l] * dims[l + 1] + dims[l + 1]
            products = 4 * rows[l + 1] * dims[l] * dims[l + 1] + edges[l] * dims[l]
        # backward: the weight gradient, and above the bottom layer the input gradient
        flops += products * (1 if not back else 2 if l == 0 else 3)
    total += rows[0] * dims[0] * el + params * 4 * (2 if back else 1) + c["batch"] * dims[-1] * 4
    return {"bytes": total, "flops": flops}


def _cost(c):
    w = work(c)
    return max(w["bytes"], w["flops"] / 50)


def tolerance(case):
    """About four times the largest difference seen between the library and the same model in 64-bit sums
    (with the bf16 roundings of what is stored), over several seeds of every listed case and 40 drawn ones;
    the same model in torch float32 shows the same sizes."""
    c = dict(_BASE, **case)
    if c["kind"] in ("group", "presample", "cached"):
        return "exact"                              # ids, counts and copied rows
    if c["dtype"] == "bf16":
        if c["kind"] == "infer":
            return {"rel": 6e-4, "max": 4e-2}       # seen 1.3e-4, 9e-3: a stored activation rounds the other way
        return {"rel": 1.5e-2, "max": 0.15}         # seen 3.8e-3, 3.6e-2: that, and ReLU decisions
    if c["kind"] == "infer":
        return {"rel": 2.4e-6, "max": 1.4e-5}       # seen 5.9e-7, 3.3e-6
    if c["kind"] == "gat":
        return {"rel": 1.6e-5, "max": 1.3e-4}       # seen 4.8e-6, 3.2e-5
    # A pre-activation that is zero to rounding (about one in 2e7) is masked either way by the ReLU's
    # derivative, and its row's whole gradient with it: seen up to 3.2e-3, 5.9e-2 where there are millions
    # of them (both sides can differ from the true decision); else 9.8e-7, 6e-6
    rows, dims = _levels(c)[0], _ints(c["dims"])
    if sum(r * d for r, d in zip(rows[1:-1], dims[1:-1])) > 200_000:
        return {"rel": 1.2e-2, "max": 0.24}
    return {"rel": 4e-6, "max": 2.4e-5}
