"""Performance cases of the library: what its users have it do, over the sizes
the tests, the benchmark and the served form use.

Graphs are the two families of the repository's recipes (synth): R-MAT
(0.57, 0.19, 0.19, 0.05; power law, no ID permutation) and random geometric
graphs in the unit square or cube (IDs ordered by grid cell), drawn here on
the GPU from the seed alone so that inputs take little time to make.
"""
from __future__ import annotations

import math

import torch

import paper_2410_19119_amd as lp


# ------------------------------------------------------------------ inputs --

def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7FFFFFFFFFFF)
    return g


def _csr(n, keys):
    """CSR (int64 offsets, int32 neighbours) of sorted distinct keys u * n + v."""
    u = torch.div(keys, n, rounding_mode="floor")
    adj = (keys - u * n).to(torch.int32)
    xadj = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    xadj[1:] = torch.cumsum(torch.bincount(u, minlength=n), 0)
    return xadj, adj


def _both_ways(n, keys):
    """CSR of the undirected edges u * n + v, u < v."""
    u = torch.div(keys, n, rounding_mode="floor")
    return _csr(n, torch.sort(torch.cat([keys, (keys - u * n) * n + u]))[0])


def _rmat(n, ef, seed):
    """R-MAT over n IDs (2^ceil(log2 n) cells, larger endpoints rejected); every
    seed gives the same number of edges (0.9 ef n), so that outputs of all
    seeds have one size."""
    scale = max(1, math.ceil(math.log2(n)))
    gen = _gen(seed, 1)
    want = int(0.9 * ef * n)
    got = None
    while got is None or got.numel() < want:
        parts = [] if got is None else [got]
        left = ef * n if got is None else max(1024, ef * n // 4)
        while left > 0:
            m = min(left, 1 << 25)
            left -= m
            u = torch.zeros(m, dtype=torch.int64, device="cuda")
            v = torch.zeros(m, dtype=torch.int64, device="cuda")
            for _ in range(scale):
                r = torch.rand(m, device="cuda", generator=gen)
                u.mul_(2).add_(r >= 0.76)
                v.mul_(2).add_(((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
            keep = (u != v) & (u < n) & (v < n)
            u, v = u[keep], v[keep]
            parts.append(torch.minimum(u, v) * n + torch.maximum(u, v))
        got = torch.unique(torch.cat(parts))
    extra = got.numel() - want
    if extra:  # drop the surplus evenly
        keep = torch.ones(got.numel(), dtype=torch.bool, device="cuda")
        keep[torch.arange(extra, device="cuda") * got.numel() // extra] = False
        got = got[keep]
    return _both_ways(n, got)


def _rgg(dim, n, deg, seed):
    """Random geometric graph with n deg / 2 edges (the closest pairs), IDs
    ordered by grid cell, then x."""
    wide = 1.6 * deg  # pairs are collected somewhat further than needed
    r = math.sqrt(wide / (math.pi * (n - 1))) if dim == 2 else (3.0 * wide / (4.0 * math.pi * (n - 1))) ** (1.0 / 3.0)
    side = max(1, int(1.0 / r))
    gen = _gen(seed, 2)
    p = torch.rand(n, dim, device="cuda", dtype=torch.float64, generator=gen)
    c = torch.clamp((p * side).to(torch.int64), max=side - 1)
    cell = c[:, 0]
    for k in range(1, dim):
        cell = cell * side + c[:, k]
    order = torch.argsort(p[:, 0])
    order = order[torch.argsort(cell[order], stable=True)]
    p, c, cell = p[order], c[order], cell[order]
    start = torch.zeros(side ** dim + 1, dtype=torch.int64, device="cuda")
    start[1:] = torch.cumsum(torch.bincount(cell, minlength=side ** dim), 0)
    ids = torch.arange(n, device="cuda")
    keys, dist = [], []
    rows = [(a,) for a in (-1, 0, 1)] if dim == 2 else [(a, b) for a in (-1, 0, 1) for b in (-1, 0, 1)]
    for off in rows:  # a row of up to three cells, contiguous in the last coordinate
        ok = torch.ones(n, dtype=torch.bool, device="cuda")
        row = torch.zeros(n, dtype=torch.int64, device="cuda")
        for k, o in enumerate(off):
            x = c[:, k] + o
            ok &= (x >= 0) & (x < side)
            row = row * side + x
        row = torch.where(ok, row, 0) * side
        lo = start[row + torch.clamp(c[:, dim - 1] - 1, min=0)]
        hi = start[row + torch.clamp(c[:, dim - 1] + 1, max=side - 1) + 1]
        lo = torch.maximum(lo, ids + 1)  # u < v
        cnt = torch.where(ok, torch.clamp(hi - lo, min=0), 0)
        step = 1 << 20
        for a in range(0, n, step):
            k = cnt[a:a + step]
            u = torch.repeat_interleave(ids[a:a + step], k)
            first = torch.cumsum(k, 0) - k
            v = torch.arange(u.numel(), device="cuda") - torch.repeat_interleave(first - lo[a:a + step], k)
            d = ((p[u] - p[v]) ** 2).sum(1)
            near = d <= r * r
            keys.append(u[near] * n + v[near])
            dist.append(d[near])
    keys = torch.cat(keys)[torch.argsort(torch.cat(dist))[: n * deg // 2]]
    return _both_ways(n, keys)


def _edge_weights(xadj, adj, seed):
    """Symmetric weights 1..100 from a hash of the endpoint pair."""
    u = torch.repeat_interleave(torch.arange(xadj.numel() - 1, device="cuda"), xadj[1:] - xadj[:-1])
    v = adj.to(torch.int64)
    h = torch.minimum(u, v) * 0x9E3779B1 + torch.maximum(u, v) * 0x85EBCA6B + int(seed) * 0x27D4EB2F
    return (((h ^ (h >> 15)) % 100 + 100) % 100 + 1).to(torch.int32)


def _inputs(case, seed):
    """(n, xadj, adjncy, adjwgt or None, vwgt or None) on the GPU."""
    n, deg = case["n"], case["deg"]
    xadj, adj = _rmat(n, deg, seed) if case["graph"] == "rmat" else _rgg(2 if case["graph"] == "rgg2d" else 3, n, deg, seed)
    w = vw = None
    if case["weights"]:
        w = _edge_weights(xadj, adj, seed)
        vw = torch.randint(1, 8, (n,), dtype=torch.int32, device="cuda", generator=_gen(seed, 3))
    return n, xadj, adj, w, vw


def _handle(case, csr):
    if case["format"] == "plain":
        return lp.lp_graph_from_csr(*csr)
    return lp.lp_compress(*csr, intervals=case["format"] == "itv")


def _batch_sizes(case):
    """Uneven graphs, n spread log-uniformly over [1e3, nmax], every other one R-MAT."""
    span = math.log(case["n"] / 1e3)
    return [("rmat" if i % 2 else "rgg2d", int(1e3 * math.exp(span * ((i + 1) * 0.6180339887 % 1.0))))
            for i in range(case["graphs"])]


def _zeros(*sizes):
    return [torch.zeros(k, dtype=t, device="cuda") for k, t in sizes]


def _into(bufs, outs):
    """The outputs in a program's own buffers, whose size does not depend on the result's."""
    for b, o in zip(bufs, outs):
        b[: o.numel()].copy_(o)
    return list(bufs)


# ------------------------------------------------------------------- cases --

def listed():
    def c(name, op, graph, n, deg, fmt="gap", weights=False, **more):
        return dict(name=name, op=op, graph=graph, n=n, deg=deg, format=fmt, weights=weights, **more)

    return [
        # the small clustering of the parity tests: latency and launches
        c("cluster_rgg2d_16k", "cluster", "rgg2d", 16384, 8, cap=32, rounds=5, calls=0),
        # the large one, on a handle that a program clusters again and again
        # (it holds its degree-ordered copy by then)
        c("cluster_rmat24", "cluster", "rmat", 1 << 24, 16, cap=256, rounds=5, calls=2),
        # a weighted plain graph, as every coarse level is
        c("cluster_plain_700k", "cluster", "rmat", 700001, 12, fmt="plain", weights=True, cap=1000, rounds=5, calls=0),
        # compression of a caller's CSR: power law, and weighted geometric with intervals
        c("compress_rmat23", "compress", "rmat", 1 << 23, 16),
        c("compress_itv_rgg3d_1m", "compress", "rgg3d", 1000003, 27, fmt="itv", weights=True),
        # back to CSR
        c("decompress_rmat22w", "decompress", "rmat", 3000017, 16, weights=True),
        # one coarsening step's contraction (labels of a clustering)
        c("contract_rmat23", "contract", "rmat", 1 << 23, 16, cap=256),
        # the objective of a clustering
        c("cut_rmat22", "cut", "rmat", 1 << 22, 16, cap=256),
        # refinement of a 64-way partition on the input graph
        c("refine_rmat22_k64", "refine", "rmat", 1 << 22, 16, k=64, rounds=5, gain_table=False),
        # the gain table: build, a batch of moves, queries
        c("gain_rmat21_k64", "gain", "rmat", 2000003, 16, k=64),
        # many uneven graphs in one call
        c("batch_48", "batch", "mixed", 200000, 8, graphs=48, rounds=5),
        # the whole multilevel partition (coarsening, projection, refinement on every level)
        c("partition_rgg2d_1m", "partition", "rgg2d", 1 << 20, 8, k=8, subrounds=1),
    ]


def draw(rng):
    def size(lo, hi):
        return int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) | 1

    op = rng.choice(["cluster", "cluster", "compress", "decompress", "contract", "cut", "refine", "gain", "batch", "partition"])
    if op == "batch":
        return dict(op=op, graph="mixed", n=size(2000, 200000), deg=8, format="gap", weights=False,
                    graphs=rng.randint(4, 48), rounds=5)
    graph = rng.choice(["rmat", "rmat", "rgg2d", "rgg3d"])
    deg = {"rmat": rng.randint(8, 16), "rgg2d": 8, "rgg3d": 27}[graph]
    c = dict(op=op, graph=graph, n=size(2000, {"rmat": 4000000, "rgg2d": 4000000, "rgg3d": 1000000}[graph]), deg=deg,
             format=rng.choice(["gap", "gap", "itv"] if op in ("compress", "decompress") else ["gap", "gap", "plain", "itv"]),
             weights=rng.random() < 0.35)
    if op in ("cluster", "contract", "cut"):
        c["cap"] = rng.choice([32, 256, 12288])
    if op == "cluster":
        c.update(rounds=rng.choice([3, 5]), calls=rng.choice([0, 2]))
    elif op == "refine":
        c.update(k=rng.choice([2, 8, 64]), rounds=5, gain_table=rng.random() < 0.4)
    elif op == "gain":
        c["k"] = rng.choice([2, 8, 64, 300])
    elif op == "partition":
        c.update(n=size(2000, 1000000 if graph != "rgg3d" else 400000), k=rng.choice([2, 8, 64]), subrounds=rng.choice([1, 4]))
    return c


def prepare(case, seed):
    op = case["op"]
    if op == "batch":
        gs = []
        for i, (kind, n) in enumerate(_batch_sizes(case)):
            gs.append(lp.lp_compress(n, *(_rmat(n, case["deg"], seed * 64 + i) if kind == "rmat"
                                          else _rgg(2, n, case["deg"], seed * 64 + i))))
        params = [lp.coarsen_params(g.n, g.total_vwgt)[1] for g in gs]
        return dict(case=case, graphs=gs, caps=params, seeds=[seed + i for i in range(len(gs))])
    csr = _inputs(case, seed)
    if op == "compress":
        room = (10 if case["weights"] else 5) * csr[2].numel() + 6 * csr[0]
        return dict(case=case, csr=csr, bufs=_zeros((csr[0] + 1, torch.int64), (room, torch.uint8)))
    s = dict(case=case, g=_handle(case, csr), seed=seed)
    g = s["g"]
    if op in ("contract", "cut"):
        s["labels"] = lp.lp_cluster(g, case["cap"], 5, seed, config=dict(reorder=2))
        if op == "contract":
            s["bufs"] = _zeros((g.n + 1, torch.int64), (g.two_m, torch.int32), (g.two_m, torch.int32), (g.n, torch.int32))
    elif op == "cluster":
        for _ in range(case["calls"]):
            lp.lp_cluster(g, case["cap"], 1, seed)
    elif op in ("refine", "gain"):
        s["blocks"] = lp.lp_initial_partition(g, case["k"])
    if op == "gain":
        m = max(1, g.n // 50)
        gen = _gen(seed, 4)
        s["moved"] = torch.randperm(g.n, device="cuda", generator=gen)[:m].to(torch.int32)
        s["to"] = torch.randint(0, case["k"], (m,), dtype=torch.int32, device="cuda", generator=gen)
        s["qu"] = torch.randint(0, g.n, (4 * g.n,), dtype=torch.int32, device="cuda", generator=gen)
        s["qb"] = torch.randint(0, case["k"], (4 * g.n,), dtype=torch.int32, device="cuda", generator=gen)
    return s


def run(s):
    case = s["case"]
    op = case["op"]
    if op == "cluster":
        return lp.lp_cluster(s["g"], case["cap"], case["rounds"], s["seed"])
    if op == "compress":
        g = _handle(case, s["csr"])
        out = _into(s["bufs"], lp.lp_graph_export(g))
        g.free()
        return out
    if op == "decompress":
        return lp.lp_decompress(s["g"])
    if op == "contract":
        c, mp = lp.lp_contract(s["g"], s["labels"])
        out = _into(s["bufs"], lp.lp_decompress(c)) + [mp]
        c.free()
        return out
    if op == "cut":
        return lp.lp_edge_cut(s["g"], s["labels"])
    if op == "refine":
        k = case["k"]
        return lp.lp_refine(s["g"], s["blocks"], k, lp.max_block_weight(s["g"].total_vwgt, k), case["rounds"], s["seed"],
                            config=dict(gain_table=int(case["gain_table"])))
    if op == "gain":
        t = lp.GainTable(s["g"], s["blocks"], case["k"])
        t.move(s["moved"], s["to"])
        out = t.affinity(s["qu"], s["qb"])
        t.free()
        return out
    if op == "batch":
        return lp.lp_batch_cluster(s["graphs"], s["caps"], case["rounds"], s["seeds"])
    return lp.partition(s["g"], case["k"], seed=s["seed"], subrounds=case["subrounds"], refine_subrounds=case["subrounds"])


def exact(case, seed):
    """Plain torch answers where the output has a definition that torch computes
    directly; clusterings, partitions and code bytes have none."""
    if case["op"] not in ("cut", "contract", "decompress", "gain"):
        return None
    n, xadj, adj, w, vw = _inputs(case, seed)
    w = torch.ones_like(adj) if w is None else w
    vw = torch.ones(n, dtype=torch.int32, device="cuda") if vw is None else vw
    if case["op"] == "decompress":
        return xadj, adj, w, vw
    s = prepare(case, seed)
    u = torch.repeat_interleave(torch.arange(n, device="cuda"), xadj[1:] - xadj[:-1])
    v = adj.to(torch.int64)
    if case["op"] == "gain":
        b = s["blocks"].to(torch.int64).clone()
        b[s["moved"].to(torch.int64)] = s["to"].to(torch.int64)
        k = case["k"]
        pairs, inv = torch.unique(u * k + b[v], return_inverse=True)
        sums = torch.zeros(pairs.numel() + 1, dtype=torch.int64, device="cuda").index_add_(0, inv, w.to(torch.int64))
        q = s["qu"].to(torch.int64) * k + s["qb"].to(torch.int64)
        at = torch.searchsorted(pairs, q)
        hit = pairs[torch.clamp(at, max=pairs.numel() - 1)] == q
        return torch.where(hit, sums[at], 0)
    lab = s["labels"].to(torch.int64)
    if case["op"] == "cut":
        return int(w.to(torch.int64)[lab[u] != lab[v]].sum().item()) // 2
    names, mp = torch.unique(lab, return_inverse=True)
    nc = names.numel()
    a, b = mp[u], mp[v]
    out = a != b
    pairs, inv = torch.unique(a[out] * nc + b[out], return_inverse=True)
    cw = torch.zeros(pairs.numel(), dtype=torch.int64, device="cuda").index_add_(0, inv, w[out].to(torch.int64))
    cx, ca = _csr(nc, pairs)
    cv = torch.zeros(nc, dtype=torch.int64, device="cuda").index_add_(0, mp, vw.to(torch.int64))
    return _into(s["bufs"], (cx, ca, cw.to(torch.int32), cv.to(torch.int32))) + [mp.to(torch.int32)]


def work(case):
    """Bytes one pass cannot do without: the graph read once (once per LP round,
    since every round needs the labels of the one before), outputs written once."""
    n, op = case["n"], case["op"]
    if op == "batch":
        span = math.log(n / 1e3)
        total = case["graphs"] * (n - 1e3) / span  # mean of the log-uniform sizes
        return {"bytes": case["rounds"] * total * (1.5 * 8 * 1.4 + 12) + 4 * total, "flops": 0}
    edges = n * (2 * case["deg"] * 0.9 if case["graph"] == "rmat" else case["deg"])  # directed
    per = (4.0 if case["format"] == "plain" else 2.0) + ((4.0 if case["format"] == "plain" else 1.5) if case["weights"] else 0)
    code = edges * per + 8 * n
    csr = edges * (8 if case["weights"] else 4) + 8 * n
    if op == "cluster" or op == "refine":
        b = case["rounds"] * (code + 12 * n)
    elif op == "compress":
        b = csr + code
    elif op == "decompress":
        b = code + edges * 8 + 12 * n
    elif op == "contract":
        b = code + 8 * n + edges * 0.9 * 8
    elif op == "cut":
        b = code + 4 * n
    elif op == "gain":
        b = code + 4 * n + 4 * n * 16
    else:
        b = 5 * 2 * case["subrounds"] * (code + 12 * n)
    return {"bytes": b, "flops": 0}
