"""The workloads that the speed of this framework is judged by.

A case is one thing a training program has the framework do, through the entry points of
`paper_2511_20564_amd.device`.  Five kinds, named in the case's "kind":

  propagate   K layers of A^ H forward and backward on a graph that stays resident (LightGCN training)
  ssl         the self-supervised branch on a resident graph: all K layers, their mean, the
              reconstruction loss, its gradient back through every layer, and the gradient's norm
  build       a graph made ready from its interaction log (pairs -> CSR -> degrees and schedule); with
              edge strengths also the values and the table that neighbour sampling reads
  minibatch   one whole training step on a freshly sampled two-hop subgraph: sample, build, look the
              feature rows up, layers with their dense update forward, and backward
  dense       the dense update H = relu(P W) alone, forward and backward (a user whose aggregation is
              elsewhere, or the head of the network)

Sizes are those of `workloads/graphs.py` (its five configurations), of the tests and of bench.py, or
lie between them.  Graphs are power-law bipartite graphs as in `workloads/graphs.py`, generated on the
GPU because they are made many times.
"""
import math

import numpy as np
import torch

import paper_2511_20564_amd.device as e2eg
from paper_2511_20564_amd import binding as B

_DEV = "cuda"


def listed():
    return [
        # configuration 1: the smallest graph anybody trains on; a step is a handful of short kernels
        dict(name="propagate_tiny", kind="propagate", n_users=2_000, n_items=1_000, n_edges=20_000, zipf=0.0,
             item_cap=0, weighted=False, dtype="f32", F=64, K=2),
        # configuration 2: a medium catalogue in fp32
        dict(name="propagate_medium", kind="propagate", n_users=100_000, n_items=50_000, n_edges=2_000_000, zipf=1.0,
             item_cap=0, weighted=False, dtype="f32", F=64, K=3),
        # edge strengths, odd sizes, rows of 144 bytes that are no multiple of a cache line
        dict(name="propagate_weighted_ragged", kind="propagate", n_users=311_027, n_items=98_507, n_edges=7_000_003,
             zipf=1.05, item_cap=0, weighted=True, dtype="bf16", F=72, K=2),
        # configuration 3: bench.py's headline workload
        dict(name="propagate_large", kind="propagate", n_users=1_000_000, n_items=500_000, n_edges=50_000_000, zipf=1.1,
             item_cap=0, weighted=False, dtype="bf16", F=128, K=3),
        # configuration 5: the largest graph that is run on one GPU
        dict(name="propagate_xlarge", kind="propagate", n_users=10_000_000, n_items=2_000_000, n_edges=500_000_000,
             zipf=1.1, item_cap=100_000, weighted=False, dtype="bf16", F=64, K=3),
        # the self-supervised branch of a training step, on a graph between configurations 2 and 3
        dict(name="ssl_branch", kind="ssl", n_users=250_007, n_items=120_011, n_edges=10_000_019, zipf=1.1, item_cap=0,
             weighted=False, dtype="bf16", F=128, K=3),
        # a log of configuration 3's size turned into a graph, as at the start of a day's training
        dict(name="build_large", kind="build", n_users=1_000_000, n_items=500_000, n_edges=50_000_000, zipf=1.1,
             item_cap=0, weighted=False),
        # a medium log with edge strengths, made ready for training and for importance sampling
        dict(name="build_weighted", kind="build", n_users=100_000, n_items=50_000, n_edges=2_000_000, zipf=1.0,
             item_cap=0, weighted=True),
        # configuration 4: bench.py's mini-batch step (uniform sampling, two layers with 128 x 128 weights)
        dict(name="minibatch_step", kind="minibatch", n_users=1_000_000, n_items=500_000, n_edges=50_000_000, zipf=1.1,
             item_cap=0, n_seeds=4096, fan0=25, fan1=10, sage=False, F=128),
        # importance-sampled GraphSAGE step with the smaller batch of a medium catalogue
        dict(name="minibatch_sage", kind="minibatch", n_users=100_000, n_items=50_000, n_edges=2_000_000, zipf=1.0,
             item_cap=0, n_seeds=1000, fan0=25, fan1=15, sage=True, F=64),
        # the dense update of a mini-batch (bench.py)
        dict(name="dense_minibatch", kind="dense", n=200_000, Fin=128, Fout=128, relu=True),
        # the same over every node of a large graph, CONCAT input, a ragged number of rows
        dict(name="dense_large", kind="dense", n=3_000_017, Fin=256, Fout=128, relu=True),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, lo, hi):
    n_edges = _log_uniform(rng, lo, hi)
    n_users = max(400, int(n_edges / rng.uniform(8, 50)))
    n_items = max(200, int(n_users * rng.uniform(0.2, 0.6)))
    return dict(n_users=n_users, n_items=n_items, n_edges=n_edges, zipf=round(rng.uniform(0.9, 1.1), 3),
                item_cap=100_000 if n_edges > 100_000_000 else 0)


def draw(rng):
    kind = rng.choice(["propagate", "propagate", "propagate", "ssl", "build", "build", "minibatch", "minibatch", "dense"])
    c = dict(kind=kind)
    if kind in ("propagate", "ssl"):
        c.update(_draw_graph(rng, 20_000, 300_000_000 if kind == "propagate" else 50_000_000))
        c.update(weighted=kind == "propagate" and rng.random() < 0.3, dtype=rng.choice(["f32", "bf16"]),
                 K=rng.choice([1, 2, 3, 4]))
        # widths of every multiple the storage type allows; the widest only where the graph leaves room
        widest = 256 if c["n_edges"] < 20_000_000 else 128 if c["n_edges"] < 80_000_000 else 64
        step = 4 if c["dtype"] == "f32" else 8
        if c["dtype"] == "f32" and c["n_edges"] >= 20_000_000:
            widest //= 2
        c["F"] = step * rng.randint(16 // step, widest // step) if rng.random() < 0.5 else rng.choice([32, 64, widest])
    elif kind == "build":
        c.update(_draw_graph(rng, 20_000, 100_000_000))
        c["weighted"] = c["n_edges"] < 60_000_000 and rng.random() < 0.4
    elif kind == "minibatch":
        c.update(_draw_graph(rng, 200_000, 50_000_000))
        c.update(n_seeds=min(_log_uniform(rng, 128, 8192), c["n_users"] // 4), fan0=rng.randint(5, 25),
                 fan1=rng.randint(5, 15), sage=rng.random() < 0.5, F=rng.choice([64, 128]))
    else:
        c.update(n=_log_uniform(rng, 1_000, 3_000_000), Fin=32 * rng.randint(1, 8), Fout=32 * rng.randint(1, 8),
                 relu=rng.random() < 0.7)
    return c


# ---- inputs --------------------------------------------------------------------------------------
def _item_cdf(n_items, zipf, n_edges, item_cap):
    """Cumulative popularity over ranks; item_cap > 0 flattens the head so that the most popular item
    expects about that many edges (workloads/graphs.py does the same)."""
    w = torch.arange(1, n_items + 1, dtype=torch.float64, device=_DEV).pow_(-zipf)
    if item_cap and n_edges / float(w.sum()) > item_cap:
        lo, hi = float(w[-1]), 1.0
        for _ in range(40):
            c = 0.5 * (lo + hi)
            if n_edges * c / float(w.clamp(max=c).sum()) > item_cap:
                hi = c
            else:
                lo = c
        w.clamp_(max=0.5 * (lo + hi))
    cdf = torch.cumsum(w, 0)
    return cdf / cdf[-1]


def _edges(c, gen):
    """Exactly c["n_edges"] distinct (user, item) pairs in random order: log-normal user activity, every
    user drawing items from the popularity without replacement (draws that repeat are made again; after
    some rounds, where the popular items of a user are used up, uniformly)."""
    nu, ni, ne = c["n_users"], c["n_items"], c["n_edges"]
    raw = torch.exp(torch.randn(nu, device=_DEV, generator=gen, dtype=torch.float32) + 2.5)
    top = min(2000, ni // 2)
    deg = torch.round(raw * (ne / float(raw.double().sum()))).long().clamp_(1, top)
    del raw
    while True:
        diff = ne - int(deg.sum())
        if diff == 0:
            break
        free = torch.nonzero(deg < top if diff > 0 else deg > 1).flatten()
        pick = free[torch.randperm(free.numel(), device=_DEV, generator=gen)[:abs(diff)]]
        deg[pick] += 1 if diff > 0 else -1
    cdf = _item_cdf(ni, c["zipf"], ne, c["item_cap"])
    item_of_rank = torch.randperm(ni, device=_DEV, generator=gen)
    ids = torch.arange(nu, device=_DEV)
    first = torch.arange(nu + 1, device=_DEV) * ni
    keys = torch.empty(0, dtype=torch.int64, device=_DEV)
    need = deg
    for rnd in range(64):
        u = torch.repeat_interleave(ids, need)
        if u.numel() == 0:
            break
        if rnd < 6:
            r = torch.rand(u.numel(), device=_DEV, generator=gen, dtype=torch.float64)
            r = item_of_rank[torch.searchsorted(cdf, r, right=True).clamp_(max=ni - 1)]
        else:
            r = torch.randint(0, ni, (u.numel(),), device=_DEV, generator=gen)
        u.mul_(ni).add_(r)
        del r
        keys = torch.unique(torch.cat([keys, u]))
        del u
        need = deg - torch.diff(torch.searchsorted(keys, first))
    keys = keys[torch.randperm(keys.numel(), device=_DEV, generator=gen)]
    items = (keys % ni).int()
    return keys.div_(ni, rounding_mode="floor").int(), items


def _strengths(n_edges, gen):
    """Interaction strengths: most near 1, a few strong (workloads.make_edge_weights)."""
    return torch.exp(torch.randn(n_edges, device=_DEV, generator=gen) * 0.8).clamp_(0.05, 50.0)


def _rows(n, F, std, dtype, gen):
    return (torch.randn(n, F, device=_DEV, generator=gen) * std).to(torch.float32 if dtype == "f32" else torch.bfloat16)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device=_DEV).manual_seed(seed)
    if c["kind"] == "dense":
        return dict(case=c, P=_rows(c["n"], c["Fin"], 0.1, "bf16", gen), gH=_rows(c["n"], c["Fout"], 1.0, "bf16", gen),
                    W=_rows(c["Fin"], c["Fout"], c["Fin"] ** -0.5, "bf16", gen))
    users, items = _edges(c, gen)
    n = c["n_users"] + c["n_items"]
    if c["kind"] == "build":
        return dict(case=c, users=users, items=items, weights=_strengths(c["n_edges"], gen) if c["weighted"] else None)
    if c["kind"] == "minibatch":
        # resident: the whole graph, its sampling table, the feature table, the weights of the layers.
        # New with every step: the seed users, the sampler's seed, the gradient that comes from the loss.
        if c["sage"]:
            g = e2eg.build_weighted_graph(c["n_users"], c["n_items"], users, items, _strengths(c["n_edges"], gen))
            table = e2eg.sampler_table(g, beta=1.5)
        else:
            g = e2eg.build_graph(c["n_users"], c["n_items"], users, items)
            table = e2eg.sampler_table(g, p=torch.ones(g.nnz, dtype=torch.float32, device=_DEV))
        fan = [c["fan0"], c["fan1"]]
        seeds = torch.randperm(c["n_users"], device=_DEV, generator=gen)[:c["n_seeds"]].sort()[0].int()
        rows = min(n, c["n_seeds"] + B.e2eg_sample_capacity(n, c["n_seeds"], fan))
        F = c["F"]
        fin = 2 * F if c["sage"] else F
        return dict(case=c, graph=g, table=table, fan=fan, seeds=seeds, draw=seed, X=_rows(n, F, 0.1, "bf16", gen),
                    g_up=_rows(rows, F, 1.0, "bf16", gen), gX=torch.zeros(rows, F, dtype=torch.bfloat16, device=_DEV),
                    W=[_rows(fin, F, fin ** -0.5, "bf16", gen) for _ in range(2)])
    if c["weighted"]:
        g = e2eg.build_weighted_graph(c["n_users"], c["n_items"], users, items, _strengths(c["n_edges"], gen))
    else:
        g = e2eg.build_graph(c["n_users"], c["n_items"], users, items)
    return dict(case=c, graph=g, X0=_rows(n, c["F"], 0.1, c["dtype"], gen),
                gY=_rows(n, c["F"], 1.0, c["dtype"], gen) if c["kind"] == "propagate" else None)


# ---- one pass ------------------------------------------------------------------------------------
def run(state):
    return _RUN[state["case"]["kind"]](state)


def _propagate(s):
    K = s["case"]["K"]
    return e2eg.propagate_fwd(s["graph"], s["X0"], K), e2eg.propagate_bwd(s["graph"], s["gY"], K)


def _ssl(s):
    g, X0, K = s["graph"], s["X0"], s["case"]["K"]
    H = e2eg.propagate_fwd(g, X0, K, all_layers=True)
    Y = e2eg.readout_mean(X0, H)
    loss, gY = e2eg.gfae_loss(X0, Y, grad_scale=1.0 / (K + 1))
    gX0 = e2eg.propagate_bwd(g, gY, K, g_shared=gY)
    return loss, Y, gX0, e2eg.block_norms(gX0, 1)


def _build(s):
    c = s["case"]
    if not c["weighted"]:
        g = e2eg.build_graph(c["n_users"], c["n_items"], s["users"], s["items"])
        return g.row_ptr, g.col_idx, g.deg, g.dinv_sqrt
    g = e2eg.build_weighted_graph(c["n_users"], c["n_items"], s["users"], s["items"], s["weights"])
    table = e2eg.sampler_table(g, beta=1.5)
    # the table is the nnz + 1 running sums of 64 bits
    return g.row_ptr, g.col_idx, g.deg, g.val, g.deg_w, g.dinv_sqrt, table[:8 * (g.nnz + 1)].view(torch.int64)


def _minibatch(s):
    c, W = s["case"], s["W"]
    sub = e2eg.sample_subgraph(s["graph"], s["table"], s["seeds"], s["fan"], s["draw"], with_weights=False)
    gs = e2eg.build_graph(sub["n_users"], sub["n_items"], sub["users"], sub["items"], add_self_loops=not c["sage"])
    H0 = s["X"].index_select(0, sub["nodes"].long())
    gW, H = (_sage_layers if c["sage"] else _gcn_layers)(gs, H0, W, s["g_up"][:gs.n], c["F"], s["gX"][:gs.n])
    # the seed users' rows are what the batch is for; the features' gradient fills the front of its buffer
    at = torch.searchsorted(sub["nodes"], s["seeds"])
    return gs.n_users, gs.n_items, gs.nnz, H.index_select(0, at), s["gX"], gW


def _gcn_layers(gs, H0, W, gH, F, gX):
    """P = A^ H, H' = relu(P W); no ReLU behind the last layer."""
    P, H = [], [H0]
    for l in range(2):
        P.append(e2eg.propagate_fwd(gs, H[l], 1))
        H.append(e2eg.layer_transform_fwd(P[l], W[l], relu=l == 0))
    grads = [None, None]
    for l in (1, 0):
        gP, grads[l] = e2eg.layer_transform_bwd(P[l], W[l], H[l + 1], gH, relu=l == 0)
        gH = e2eg.propagate_bwd(gs, gP, 1, out=None if l else gX)
    return grads, H[2]


def _sage_layers(gs, H0, W, gH, F, gX):
    """h' = relu(W . CONCAT(h, mean of the sampled neighbours)); the mean lands in the CONCAT buffer."""
    P, H = [], [H0]
    for l in range(2):
        cat = torch.empty((gs.n, 2 * F), dtype=torch.bfloat16, device=H0.device)
        cat[:, :F] = H[l]
        e2eg.aggregate(gs, H[l], B.E2EG_AGG_MEAN, out=cat[:, F:])
        P.append(cat)
        H.append(e2eg.layer_transform_fwd(cat, W[l], relu=l == 0))
    grads = [None, None]
    for l in (1, 0):
        gP, grads[l] = e2eg.layer_transform_bwd(P[l], W[l], H[l + 1], gH, relu=l == 0)
        gH = e2eg.aggregate(gs, gP[:, F:], B.E2EG_AGG_MEAN_T, addend=gP[:, :F], out=None if l else gX)
    return grads, H[2]


def _dense(s):
    c = s["case"]
    H = e2eg.layer_transform_fwd(s["P"], s["W"], relu=c["relu"])
    gP, gW = e2eg.layer_transform_bwd(s["P"], s["W"], H, s["gH"], relu=c["relu"])
    return H, gP, gW


_RUN = {"propagate": _propagate, "ssl": _ssl, "build": _build, "minibatch": _minibatch, "dense": _dense}


# ---- what a pass cannot do without ---------------------------------------------------------------
def _subgraph_size(c):
    """Expected nodes, picks and distinct pairs of a sampled subgraph (the popular items are drawn by
    several seed users; the users of the second hop hardly repeat)."""
    p = np.arange(1, c["n_items"] + 1, dtype=np.float64) ** -c["zipf"]
    p /= p.sum()
    d0 = min(c["fan0"], c["n_edges"] / c["n_users"])
    items = float((-np.expm1(-p * c["n_seeds"] * d0)).sum())
    picks1 = items * min(c["fan1"], c["n_edges"] / c["n_items"])
    users = c["n_seeds"] + c["n_users"] * -math.expm1(-picks1 / c["n_users"])
    return users + items, c["n_seeds"] * d0 + picks1


def work(case):
    c = case
    if c["kind"] == "dense":
        n, Fi, Fo = c["n"], c["Fin"], c["Fout"]
        # forward: P, W in, H out; backward: P, W, H, gH in, gP, gW out
        return dict(bytes=2 * n * (3 * Fi + 3 * Fo) + 2 * 2 * Fi * Fo + 4 * Fi * Fo, flops=6 * n * Fi * Fo)
    n, ne = c["n_users"] + c["n_items"], c["n_edges"]
    nnz = 2 * ne + n
    if c["kind"] == "build":
        # pairs in; row pointers, columns, degrees and their scales out, and the schedule's copy of the
        # structure (columns, their node ids and scales); weighted: strengths in, values out twice, table out
        each = 16 if not c["weighted"] else 16 + 4 + 4 + 8
        return dict(bytes=(12 if c["weighted"] else 8) * ne + each * nnz + 24 * n, flops=0)
    if c["kind"] == "minibatch":
        m, picks = _subgraph_size(c)
        z = 2 * picks + (0 if c["sage"] else m)
        F = c["F"]
        fin = 2 * F if c["sage"] else F
        # per pick one table entry and the pair; the subgraph's columns; feature rows in, output and
        # gradient in and out once (layers in between could stay on the chip, and are not counted)
        return dict(bytes=24 * picks + 4 * z + 2 * m * F * 4, flops=2 * (6 * m * fin * F + 2 * z * F))
    b = 2 if c["dtype"] == "bf16" else 4
    graph = nnz * (8 if c["weighted"] else 4) + 8 * n
    rows = n * c["F"] * b
    flops = 2 * c["K"] * nnz * c["F"] * (2 if c["weighted"] else 1)
    if c["kind"] == "ssl":
        # features in; the mean and the gradient with respect to the features out; the graph each way
        return dict(bytes=2 * graph + 3 * rows, flops=flops + n * c["F"] * (c["K"] + 6))
    return dict(bytes=2 * graph + 4 * rows, flops=flops)


def tolerance(case):
    if case["kind"] == "build":
        # structure, degrees and the table are whole numbers; d~ is a sum in double, rounded to fp32 once
        return {"rel": 1e-7, "max": 2.5e-7, "differ": 0.0} if case["weighted"] else "exact"
    if case["kind"] == "propagate" and case["dtype"] == "f32":
        return {"rel": 1e-5}
    if case["kind"] == "ssl" and case["dtype"] == "f32":
        return {"rel": 1e-5}
    # one rounding to bf16 per stored layer and per pre-scaled intermediate
    return {"rel": 1e-2}
