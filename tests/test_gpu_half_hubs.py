"""Whole hubs of at most half size in a launch of their own: without larger ones
(one more than the compute units) and next to a few or many, with degrees at the
bounds of the size with and without edge weights. Against the oracle: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

POOL = 16100
CASES = {"alone": ([4097, 5000, 5999, 6000], 260, []), "alone-wide": ([4097, 7999, 8000], 260, []),
         "one-launch": ([4097, 6000], 255, []), "beside": ([4097, 4099], 1030, [8001, 10001, 12000, 16000]),
         "beside-many": ([4097, 4099], 450, [8001, 10001] * 225)}


@pytest.fixture(scope="module", params=[(c, w) for c in CASES for w in (False, True) if (c, w) != ("alone-wide", True)],
                ids=lambda p: p[0] + ("-weighted" if p[1] else ""))
def graph(request, synth_mod):
    degrees, hubs, larger = CASES[request.param[0]]
    rng = np.random.default_rng(5)
    deg = np.concatenate([np.resize(degrees, hubs), larger]).astype(np.int64)
    hub = np.repeat(np.arange(len(deg)), deg)
    start = rng.integers(0, POOL, len(deg))
    leaf = len(deg) + np.concatenate([(s + 11 * np.arange(d)) % POOL for s, d in zip(start, deg)])
    src, dst = np.concatenate([hub, leaf]), np.concatenate([leaf, hub])
    o = np.lexsort((dst, src))
    n = len(deg) + POOL
    w = np.tile(rng.integers(1, 50, hub.size), 2)[o].astype(np.int32) if request.param[1] else None
    xadj = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.uint64)
    return synth_mod.Graph(n, xadj, dst[o].astype(np.int32), w)


@pytest.mark.parametrize("fmt", ["gap", "plain", "intervals"])
def test_half_size_hubs(lp, oracle_mod, graph, fmt):
    g = graph
    x = g.xadj.view(np.int64)
    if fmt == "plain":
        G = lp.lp_graph_from_csr(g.n, x, g.adjncy, g.adjwgt)
    else:
        G = lp.lp_compress(g.n, x, g.adjncy, g.adjwgt, intervals=fmt == "intervals")
    exp, _ = oracle_mod.lp_cluster(g, 300, 3, 7)
    got = lp.lp_cluster(G, 300, 3, 7)
    assert np.array_equal(got.cpu().numpy(), exp)
    assert lp.lp_edge_cut(G, exp) == oracle_mod.edge_cut(g, exp)
    C, cmap = lp.lp_contract(G, exp)
    ec, emap = oracle_mod.contract(g, exp)
    cx, ca, cw = (t.cpu().numpy() for t in lp.lp_decompress(C)[:3])
    assert np.array_equal(cmap.cpu().numpy(), emap) and np.array_equal(cx, ec.xadj.astype(np.int64))
    assert np.array_equal(ca, ec.adjncy) and np.array_equal(cw, ec.adjwgt)
