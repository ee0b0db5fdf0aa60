"""The codec takes a CSR in stretches of 2048 positions (decompression: 1664) of
the merged sequence of vertices and adjacency entries (vertex u at xadj[u] + u,
its entries after it). Stars whose centre lies right before, on and after a stretch's end, whose
neighbourhoods end there, and whose chunked records start, continue and end in
stretches of their own; all-integer, so the tolerance is zero."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _star(synth_mod, before, iso, d, weighted, tail=0):
    """`before` leaves, `iso` isolated vertices, the centre (at position
    2 * before + iso), the other d - before leaves, `tail` isolated vertices."""
    c = before + iso
    leaves = list(range(before)) + list(range(c + 1, c + 1 + d - before))
    w = [1 + (i * 7919) % 100000 for i in range(d)] if weighted else None
    g = synth_mod.from_edges(c + 1 + d - before, [(c, v) for v in leaves], w)
    if tail:
        g.n += tail
        g.xadj = np.concatenate([g.xadj, np.full(tail, g.xadj[-1], dtype=np.uint64)])
    return g


CASES = [  # before, iso, degree, tail
    (1023, 0, 1500, 0),     # centre two before the end of a stretch
    (1023, 1, 1500, 0),     # the stretch's last position, all entries in the next
    (1024, 0, 1500, 0),     # the next stretch's first position
    (0, 0, 2047, 0), (0, 0, 2048, 1), (0, 0, 2049, 5000),  # entries that end at, before and after an end
    (10, 2027, 4096, 2047),
    (831, 1, 1500, 0), (831, 2, 1500, 1000), (832, 0, 1663, 1), (0, 0, 1664, 3), (0, 0, 3328, 1664),
    (831, 1, 10001, 0), (831, 2, 10500, 0), (300, 64, 11664, 1),  # 1000-entry chunks against 1664 positions
    (1023, 1, 10001, 0),    # a split record whose entries start with a stretch
    (1022, 0, 10000, 3), (500, 3, 10001, 4096), (7, 0, 25003, 1),
]


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("case", CASES)
def test_records_across_stretches(lp, oracle_mod, synth_mod, case, weighted):
    before, iso, d, tail = case
    g = _star(synth_mod, before, iso, d, weighted, tail)
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
    offs, data = lp.lp_graph_export(G)
    o, b = oracle_mod.compress(g.n, g.xadj, g.adjncy, g.adjwgt)
    assert np.array_equal(offs.cpu().numpy().view(np.uint64), o)
    assert np.array_equal(data.cpu().numpy(), b)
    x, a, w, _ = lp.lp_decompress(G)
    assert np.array_equal(x.cpu().numpy().view(np.uint64), g.xadj)
    assert np.array_equal(a.cpu().numpy(), g.adjncy)
    if weighted:
        assert np.array_equal(w.cpu().numpy(), g.adjwgt)
    # the weighted-degree maximum sets the width of the sort keys of acceptance
    P = lp.lp_graph_from_csr(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
    exp, _ = oracle_mod.lp_cluster(g, 40, 3, 5)
    for h in (G, P):
        assert np.array_equal(lp.lp_cluster(h, 40, 3, 5).cpu().numpy(), exp)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,deg,seed", [(3000, 3, 1), (5000, 40, 2), (700, 300, 3)])
def test_long_codes_and_windows(lp, synth_mod, n, deg, seed, weighted):
    # spread-out neighbours (codes of up to five bytes, so a stretch takes
    # several windows of bytes) with vertices of every degree in between
    rng = np.random.default_rng(seed)
    ids = np.sort(rng.choice(1 << 22, n, replace=False).astype(np.int64))
    u = rng.integers(0, n, n * deg // 2)
    v = rng.integers(0, n, n * deg // 2)
    e = np.unique(np.stack([np.minimum(u, v), np.maximum(u, v)], 1)[u != v], axis=0)
    w = rng.integers(1, 2**30, len(e)) if weighted else None
    g = synth_mod.from_edges(1 << 22, ids[e], w)
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
    x, a, ww, _ = lp.lp_decompress(G)
    assert np.array_equal(x.cpu().numpy().view(np.uint64), g.xadj)
    assert np.array_equal(a.cpu().numpy(), g.adjncy)
    assert np.array_equal(ww.cpu().numpy(), g.adjwgt if weighted else np.ones(g.two_m, np.int32))


def _runs_graph(synth_mod, n, seed, hub, weighted, dup=False):
    """Vertices whose neighbourhoods mix runs of consecutive IDs of every length
    with single IDs; the last vertex of a stretch is often long."""
    rng = np.random.default_rng(seed)
    edges = []
    for u in range(0, n, 37):
        v = u + 1
        while v < min(n, u + int(rng.integers(2, hub))):
            ln = int(rng.integers(1, 7))
            edges += [(u, x) for x in range(v, min(n, v + ln))]
            v += ln + int(rng.integers(1, 4))
    e = np.unique(np.array(edges, dtype=np.int64), axis=0)
    if dup:
        e = np.concatenate([e, e[::5]])
    w = rng.integers(1, 5000, len(e)) if weighted else None
    return synth_mod.from_edges(n, e, w)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("n,hub,dup", [(64, 40, False), (1500, 60, True), (6000, 3000, False), (9000, 4800, True),
                                       (14000, 9000, False)])
def test_interval_records(lp, oracle_mod, synth_mod, n, hub, dup, weighted):
    g = _runs_graph(synth_mod, n, n + hub, hub, weighted, dup)
    if n == 6000:  # a long tail of isolated vertices
        g.n += 5000
        g.xadj = np.concatenate([g.xadj, np.full(5000, g.xadj[-1], dtype=np.uint64)])
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, intervals=True)
    offs, data = lp.lp_graph_export(G)
    o, b = oracle_mod.compress(g.n, g.xadj, g.adjncy, g.adjwgt, intervals=True)
    assert np.array_equal(offs.cpu().numpy().view(np.uint64), o)
    assert np.array_equal(data.cpu().numpy(), b)
    x, a, w, _ = lp.lp_decompress(G)
    assert np.array_equal(x.cpu().numpy().view(np.uint64), g.xadj)
    assert np.array_equal(a.cpu().numpy(), g.adjncy)
    assert np.array_equal(w.cpu().numpy(), g.adjwgt if weighted else np.ones(g.two_m, np.int32))


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("case", CASES + [(1023, 1, 4000, 0), (1023, 0, 4001, 2), (500, 1, 4096, 0), (40, 5, 13002, 9)])
def test_interval_records_across_stretches(lp, oracle_mod, synth_mod, case, weighted):
    before, iso, d, tail = case
    g = _star(synth_mod, before, iso, d, weighted, tail)
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, intervals=True)
    offs, data = lp.lp_graph_export(G)
    o, b = oracle_mod.compress(g.n, g.xadj, g.adjncy, g.adjwgt, intervals=True)
    assert np.array_equal(offs.cpu().numpy().view(np.uint64), o)
    assert np.array_equal(data.cpu().numpy(), b)


@pytest.mark.parametrize("intervals", [False, True])
@pytest.mark.parametrize("a,b", [(2, 16001), (3, 10999), (5, 4001), (4, 12000), (3, 5001)])
def test_split_records_next_to_each_other(lp, oracle_mod, synth_mod, a, b, intervals):
    # hubs 0 .. a - 1 with the same b neighbours: the last chunk of one and the
    # first chunk of the next start within a chunk length of each other
    g = synth_mod.from_edges(a + b, [(h, v) for h in range(a) for v in range(a, a + b)])
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, intervals=intervals)
    offs, data = lp.lp_graph_export(G)
    o, d = oracle_mod.compress(g.n, g.xadj, g.adjncy, intervals=intervals)
    assert np.array_equal(offs.cpu().numpy().view(np.uint64), o)
    assert np.array_equal(data.cpu().numpy(), d)
