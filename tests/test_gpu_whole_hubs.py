"""Enough hubs that those of half size get a launch of their own, with degrees
at the bounds of the sizes (4097: the smallest hub, 6000 / 8000: half size with
and without edge weights, 12000 / 16000: whole). Against the oracle: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEGREES = [4097, 5000, 6000, 6001, 7999, 8000, 8001, 9999, 10001, 12000, 12001, 16000, 16001]
HUBS, POOL = 530, 16100


@pytest.fixture(scope="module", params=[False, True], ids=["unit", "weighted"])
def graph(request, synth_mod):
    rng = np.random.default_rng(3)
    deg = np.where(np.arange(HUBS) < 2 * len(DEGREES), np.resize(DEGREES, HUBS), 4097 + np.arange(HUBS) % 3)
    hub = np.repeat(np.arange(HUBS), deg)
    leaf = HUBS + np.concatenate([rng.choice(POOL, d, replace=False) for d in deg])
    src, dst = np.concatenate([hub, leaf]), np.concatenate([leaf, hub])
    o = np.lexsort((dst, src))
    n = HUBS + POOL
    w = np.tile(rng.integers(1, 50, hub.size), 2)[o].astype(np.int32) if request.param else None
    xadj = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.uint64)
    return synth_mod.Graph(n, xadj, dst[o].astype(np.int32), w)


@pytest.mark.parametrize("fmt", ["gap", "plain", "intervals"])
def test_many_whole_hubs(lp, oracle_mod, graph, fmt):
    g = graph
    x = g.xadj.view(np.int64)
    if fmt == "plain":
        G = lp.lp_graph_from_csr(g.n, x, g.adjncy, g.adjwgt)
    else:
        G = lp.lp_compress(g.n, x, g.adjncy, g.adjwgt, intervals=fmt == "intervals")
    exp, ost = oracle_mod.lp_cluster(g, 300, 3, 7)
    got, st = lp.lp_cluster(G, 300, 3, 7, stats=True)
    assert st.buckets[3] >= 520
    assert np.array_equal(got.cpu().numpy(), exp)
    assert lp.lp_edge_cut(G, exp) == oracle_mod.edge_cut(g, exp)
    C, cmap = lp.lp_contract(G, exp)
    ec, emap = oracle_mod.contract(g, exp)
    cx, ca, cw = (t.cpu().numpy() for t in lp.lp_decompress(C)[:3])
    assert np.array_equal(cmap.cpu().numpy(), emap) and np.array_equal(cx, ec.xadj.astype(np.int64))
    assert np.array_equal(ca, ec.adjncy) and np.array_equal(cw, ec.adjwgt)
