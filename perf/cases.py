"""The calls whose speed is watched, one case each, through the package's public entry points.

A case names an operation (`op`), a graph recipe (`kind`, `size`) and how many trees it takes (`count`):

  estimate  Graph.estimate: sample, number, evaluate, reduce
  trees     Graph.sample_trees with the per-vertex draw counts
  evaluate  Graph.evaluate_trees on parent arrays the caller holds
  batch     one replay of a captured launch over a grid, a road-like and a power-law graph
  update    a resident set under a deletion batch, its re-insertion, and the queries between
  query     Graph.samples_query of a resident set

Graphs are the package's own recipes: 4-neighbour grids, thinned random geometric graphs (road-like, mean
degree 2.8), Chung-Lu power laws of mean degree 10 (social) and 76 (dense).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import graphgen
import paper_2511_16356_amd as kc


def listed():
    return [
        # what a served query costs: the smallest call, where launches and copies count
        {"name": "query_grid_1024", "op": "query", "kind": "grid", "size": 4900, "count": 1024},
        # one tree of the accuracy workload's grid: latency of a call with no parallelism across samples
        {"name": "estimate_grid32_1", "op": "estimate", "kind": "grid", "size": 1024, "count": 1},
        # the accuracy workload: 2,000 trees of the 32 x 32 grid
        {"name": "estimate_grid32_2000", "op": "estimate", "kind": "grid", "size": 1024, "count": 2000},
        # a sparse graph of a served size, long walks, deep reference tree
        {"name": "estimate_road_12k_256", "op": "estimate", "kind": "road", "size": 12007, "count": 256},
        # a large sparse graph (large chain table): few samples, bound by one sample's latency
        {"name": "estimate_grid_100k_48", "op": "estimate", "kind": "grid", "size": 102400, "count": 48},
        # the power-law workload's recipe, as many samples as fill the chip
        {"name": "estimate_social_500k_2048", "op": "estimate", "kind": "social", "size": 500000, "count": 2048},
        # the dense workload's recipe (rows far longer than the inline neighbours)
        {"name": "estimate_dense_150k_2560", "op": "estimate", "kind": "dense", "size": 150001, "count": 2560},
        # trees handed to the caller, with their draw counts; fewer samples than the chip holds
        {"name": "trees_social_100k_300", "op": "trees", "kind": "social", "size": 101777, "count": 300},
        # re-evaluation of held trees, shallow reference tree (a resident set after an update, a tau0 study)
        {"name": "evaluate_social_300k_512", "op": "evaluate", "kind": "social", "size": 300007, "count": 512},
        # the same with a deep reference tree (the Fenwick sweep)
        {"name": "evaluate_road_60k_1024", "op": "evaluate", "kind": "road", "size": 60013, "count": 1024},
        # the serving mix in one captured launch
        {"name": "batch_mix_5k_200", "op": "batch", "kind": "mix", "size": 5000, "count": 200},
        # a resident set of the serving mix under improved maintenance
        {"name": "update_social_20k_1024", "op": "update", "kind": "social", "size": 20000, "count": 1024, "edges": 4,
         "improved": True},
    ]


# op -> kind -> (smallest size, largest size, smallest count, largest count, size x count limit)
RANGES = {
    "estimate": {"grid": (1024, 102400, 1, 2048, 8e6), "road": (2000, 12000, 1, 512, 3e6),
                 "social": (10000, 500000, 1, 2560, 6e8), "dense": (10000, 150000, 1, 2560, 2.5e8)},
    "trees": {"grid": (1024, 16384, 1, 1024, 6e6), "road": (2000, 10000, 1, 512, 2e6),
              "social": (10000, 200000, 1, 1024, 6e7), "dense": (10000, 100000, 1, 1024, 6e7)},
    "evaluate": {"grid": (1024, 16384, 1, 2048, 1e7), "road": (2000, 60000, 1, 1024, 2e7),
                 "social": (10000, 300000, 1, 2048, 1.5e8), "dense": (10000, 150000, 1, 2048, 1.5e8)},
    "batch": {"mix": (1500, 5000, 1, 400, 1e6)},
    "update": {"grid": (1024, 10000, 16, 1024, 1e7), "road": (2000, 8000, 16, 512, 2e6),
               "social": (5000, 40000, 16, 1024, 2e7)},
    "query": {"grid": (1024, 4900, 16, 2048, 6e6), "social": (5000, 30000, 16, 2048, 2e7)},
}
OPS = ["estimate"] * 4 + ["evaluate"] * 2 + ["trees", "batch", "update", "query"]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(OPS)
    kind = rng.choice(sorted(RANGES[op]))
    lo, hi, clo, chi, most = RANGES[op][kind]
    size = _log_uniform(rng, lo, hi)
    count = max(clo, min(_log_uniform(rng, clo, chi), int(most / size)))
    case = {"op": op, "kind": kind, "size": size, "count": count}
    if op == "update":
        case["edges"] = rng.randint(1, 8)
        case["improved"] = rng.random() < 0.5
    return case


@functools.lru_cache(maxsize=4)
def _graph(kind, size):
    if kind == "grid":
        rows = max(2, int(math.isqrt(size)))
        return graphgen.grid(rows, max(2, round(size / rows)))
    if kind == "road":
        return graphgen.road_like(size, seed=0)
    if kind == "social":
        return graphgen.chung_lu(size, 2.2, 10.0, max(50.0, size ** 0.5 * 5), seed=0)
    return graphgen.chung_lu(size, 2.0, 76.0, max(500.0, size ** 0.5 * 17), seed=0)


def _kinds(case):
    return ["grid", "road", "social"] if case["op"] == "batch" else [case["kind"]]


def prepare(case, seed):
    """The case's graph, prepared and resident with the workspace a program reserves ahead of its calls; the
    seed is that of the trees (and of the edges an update takes)."""
    op, count = case["op"], case["count"]
    host = [_graph(k, case["size"]) for k in _kinds(case)]
    graphs = [kc.Graph.from_graph(h) for h in host]
    s = {"op": op, "seed": seed, "count": count, "g": graphs[0]}
    if op == "batch":
        s["batch"] = kc.Batch(graphs, [seed + j for j in range(len(graphs))], [0] * len(graphs), [count] * len(graphs))
        return s
    graphs[0].reserve(count)
    if op == "evaluate":
        s["parents"] = graphs[0].sample_trees(seed, 0, count, popcounts=False, steps=False)[0]
    elif op in ("query", "update"):
        if case.get("improved"):
            graphs[0].set_option(kc.KC_OPT_MAINTENANCE, kc.KC_MAINT_IMPROVED)
        graphs[0].samples_init(seed, count)
    if op == "update":
        e = graphgen.deletion_batch(host[0], case["edges"], np.random.default_rng(seed))
        s["u"], s["v"] = np.array([x[0] for x in e], np.int32), np.array([x[1] for x in e], np.int32)
        s["ins"] = np.ones(len(e), np.uint8)
    return s


def _halves(x):
    return [x & ((1 << 62) - 1), x >> 62]


def _of(est):
    # the exact sums come as two 62-bit halves; the count of lock-step rounds is left out: it describes the
    # launch's schedule, on which no result depends
    return {"kappa": est.kappa, "std_error": est.std_error, "sum_f": _halves(est.sum_f), "sum_f2": _halves(est.sum_f2),
            "count": est.count, "draws": est.total_steps}


def run(s):
    g, op = s["g"], s["op"]
    if op == "estimate":
        est, f, draws = g.estimate(s["seed"], 0, s["count"], per_sample=True)
        return {"est": _of(est), "f": f, "steps": draws}
    if op == "trees":
        return list(g.sample_trees(s["seed"], 0, s["count"]))
    if op == "evaluate":
        return g.evaluate_trees(s["parents"])
    if op == "query":
        return _of(g.samples_query())
    if op == "batch":
        s["batch"].launch()
        ests, launches = s["batch"].results()
        return {"est": [_of(e) for e in ests], "f": [s["batch"].f(j) for j in range(len(ests))], "launches": launches}
    removed = g.apply_updates(s["u"], s["v"])
    without = _of(g.samples_query())
    added = g.apply_updates(s["u"], s["v"], s["ins"])
    after = _of(g.samples_query())
    parents, f, ids = g.samples_get()
    return {"removed": removed, "without": without, "added": added, "after": after, "parents": parents, "f": f,
            "ids": ids, "weights": g.samples_weights()}


def work(case):
    """Bytes: the CSR once per pass, each tree's parents written and read once where they are not the caller's,
    the outputs.  Operations: one Philox4x32-10 block (about 80 integer operations) for each vertex of a drawn
    tree, which draws at least once; about 16 per vertex to evaluate one."""
    op, count, size = case["op"], case["count"], case["size"]
    total = {"bytes": 0.0, "flops": 0.0}
    if op == "query":
        return {"bytes": 8.0 * count, "flops": 4.0 * count}
    for kind in _kinds(case):
        n = size * {"grid": 1.0, "road": 0.79, "social": 0.97, "dense": 1.0}[kind]
        csr = 8 * n + 4 * n * {"grid": 3.9, "road": 2.8, "social": 10.2, "dense": 74.0}[kind]
        trees = n * count
        if op == "trees":
            total["bytes"] += csr + 8 * trees + 8 * count
            total["flops"] += 80 * trees
        elif op == "evaluate":
            total["bytes"] += csr + 4 * trees + 8 * count
            total["flops"] += 16 * trees
        elif op == "update":  # both updates re-evaluate the whole set
            total["bytes"] += 2 * (csr + 4 * trees) + 4 * trees
            total["flops"] += 2 * 16 * trees
        else:
            total["bytes"] += csr + 8 * trees + 16 * count
            total["flops"] += 96 * trees
    return total


# ---------------------------------------------------------------- the same in plain torch

M32 = 0xFFFFFFFF


def _slots(seed, s, v, k, deg):
    """floor(x deg / 2^64), x the first two words of Philox4x32-10 on counter (k, v, s_lo, s_hi)."""
    x0, x1, x2, x3 = k & M32, v & M32, s & M32, (s >> 32) & M32
    k0, k1 = seed & M32, (seed >> 32) & M32
    for _ in range(10):
        a, b = 0xD2511F53 * x0, 0xCD9E8D57 * x2
        x0, x1, x2, x3 = ((b >> 32) & M32) ^ x1 ^ k0, b & M32, ((a >> 32) & M32) ^ x3 ^ k1, a & M32
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return (x1 * deg + ((x0 * deg) >> 32)) >> 32


def _plain_trees(off, adj, root, seed, count):
    """Cycle popping of `count` samples at once: every cycle of the current arrows is popped in each round."""
    dev = off.device
    n = off.numel() - 1
    deg = off[1:] - off[:-1]
    nxt = torch.full((count * n,), -1, dtype=torch.int64, device=dev)
    k = torch.zeros(count * n, dtype=torch.int64, device=dev)
    jump = torch.full((count * n,), -1, dtype=torch.int64, device=dev)  # -1: reaches the root
    act = torch.arange(count * n, device=dev)
    act = act[act % n != root]
    new = act
    while act.numel():
        v, s = new % n, new // n
        y = adj[off[v] + _slots(seed, s, v, k[new], deg[v])]
        nxt[new] = torch.where(y == root, -1, s * n + y)
        k[new] += 1
        # vertices whose path reaches the root are settled for good
        jump[act] = nxt[act]
        for _ in range(max(1, math.ceil(math.log2(n)))):
            j = jump[act]
            jump[act] = torch.where(j < 0, j, jump[j.clamp(min=0)])
        act = act[jump[act] >= 0]
        on = torch.zeros(count * n, dtype=torch.bool, device=dev)
        on[jump[act]] = True  # n steps on, an unsettled vertex is on a cycle
        new = act[on[act]]
    base = torch.arange(count, device=dev).repeat_interleave(n) * n
    par = torch.where(nxt < 0, root, nxt - base).view(count, n)
    par[:, root] = root
    return par, k.view(count, n).sum(1)


def _plain_f(off, adj, root, par):
    """Theorem 3.4's sums, every tree at once, over the breadth-first reference tree."""
    dev = off.device
    count, n = par.shape
    deg = (off[1:] - off[:-1])
    two_m = int(off[-1])
    src = torch.repeat_interleave(torch.arange(n, device=dev), deg)
    dist = torch.full((n,), n, dtype=torch.int64, device=dev)
    dist[root] = 0
    level = 0
    while True:
        far = adj[(dist[src] == level) & (dist[adj] == n)]
        if far.numel() == 0:
            break
        level += 1
        dist[far] = level
    up = dist[adj] == dist[src] - 1
    p0 = torch.full((n,), n, dtype=torch.int64, device=dev).scatter_reduce(0, src[up], adj[up], "amin")
    p0[root] = root
    # subtree volumes and depths by pointer doubling
    steps = max(1, math.ceil(math.log2(n))) + 1
    vol, anc = deg.repeat(count, 1), par.clone()
    live = torch.ones_like(par, dtype=torch.bool)
    live[:, root] = False
    for _ in range(steps):
        vol = vol + torch.zeros_like(vol).scatter_add(1, anc, torch.where(live, vol, 0))
        live = live & live.gather(1, anc)
        anc = anc.gather(1, anc)
    # preorder position: the offset among the siblings, summed along the path to the root
    order = par.sort(dim=1, stable=True)[1]
    in_order = torch.where(order == root, 0, vol.gather(1, order))
    before = in_order.cumsum(1) - in_order
    ps = par.gather(1, order)
    first = torch.full((count, n), 1 << 62, dtype=torch.int64, device=dev).scatter_reduce(1, ps, before, "amin")
    tin = torch.zeros_like(par).scatter(1, order, before - first.gather(1, ps)) + deg[par]
    tin[:, root] = 0
    anc = par.clone()
    for _ in range(steps):
        tin = tin + tin.gather(1, anc)
        anc = anc.gather(1, anc)
    # walk up the reference tree from every vertex
    x = torch.arange(n, device=dev)
    f = torch.zeros(count, dtype=torch.int64, device=dev)
    weight = two_m - vol
    for _ in range(level):
        z, on = p0[x], x != root
        q = torch.where((par[:, x] == z) & (tin[:, x] <= tin) & (tin < tin[:, x] + vol[:, x]), weight[:, x], 0)
        back = (par[:, z] == x) & (z != root) & (tin[:, z] <= tin) & (tin < tin[:, z] + vol[:, z])
        q = q - torch.where(back, weight[:, z], 0)
        f += (q * torch.where(on, deg, 0)).sum(1)
        x = z
    return f


def _exact_of(f, draws, two_m):
    fs = [int(x) for x in f.tolist()]
    c = len(fs)
    s1, s2 = sum(fs), sum(x * x for x in fs)
    var = (s2 * c - s1 * s1) / (c * c * (c - 1.0)) if c > 1 else math.nan
    return {"kappa": s1 / (two_m * c), "std_error": math.sqrt(var) / two_m if c > 1 else math.nan, "sum_f": _halves(s1),
            "sum_f2": _halves(s2), "count": c, "draws": None if draws is None else int(draws.sum())}


def exact(case, seed):
    """Whole numbers need no second opinion; estimates and queries do, where the plain rounds are few enough."""
    op, count, size = case["op"], case["count"], case["size"]
    kinds = _kinds(case)
    if op not in ("estimate", "batch", "query") or size * count > 2e7 or ("road" in kinds and size > 6000):
        return None
    if "grid" in kinds and size > 20000:
        return None
    ests, fs, steps = [], [], []
    for j, kind in enumerate(kinds):
        h = _graph(kind, size)
        off = torch.from_numpy(h.offsets.astype(np.int64)).cuda()
        adj = torch.from_numpy(h.indices.astype(np.int64)).cuda()
        root = int(np.argmax(np.diff(h.offsets)))
        par, draws = _plain_trees(off, adj, root, seed + j, count)
        f = _plain_f(off, adj, root, par)
        ests.append(_exact_of(f, draws, h.two_m))
        fs.append(f)
        steps.append(draws)
    if op == "batch":
        return {"est": ests, "f": fs, "launches": 1}
    if op == "query":
        return {**ests[0], "draws": None}
    return {"est": ests[0], "f": fs[0], "steps": steps[0]}
