"""Contraction by buckets of IDs and by tables: clusters at the record counts
where one size of group hands over to the next, with neighbours that all
differ, repeat a few times, or repeat so often (or lie so unevenly) that the
tables take over. Integer work against the oracle: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 2047, 2048, 2049, 5000, 17000]
POOL = 40000


@pytest.mark.parametrize("weights", [False, True])
@pytest.mark.parametrize("pattern", ["distinct", "pairs", "hot", "uneven", "one"])
def test_cluster_sizes(lp, oracle_mod, synth_mod, pattern, weights):
    # vertex i has SIZES[i] neighbours in a pool whose labels give them few or many coarse ones
    rng = np.random.default_rng(5)
    edges = []
    for i, d in enumerate(SIZES):
        edges += [(i, len(SIZES) + int(v)) for v in rng.choice(POOL, d, replace=False)]
    w = rng.integers(1, 1000, len(edges)).tolist() if weights else None
    g = synth_mod.from_edges(len(SIZES) + POOL, edges, w)
    v = np.arange(POOL)
    pool = {"distinct": v, "pairs": v // 2, "hot": np.where(v % 10 == 0, v, 7), "one": v * 0,
            "uneven": np.minimum(v, (1.3 ** (v % 40)).astype(np.int64))}[pattern]
    labels = np.concatenate([np.arange(len(SIZES)), len(SIZES) + pool]).astype(np.int32)
    exp, emap = oracle_mod.contract(g, labels)
    for make in (lp.lp_compress, lp.lp_graph_from_csr):
        G = make(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
        C, cmap = lp.lp_contract(G, labels)
        x, a, cw, vw = (t.cpu().numpy() for t in lp.lp_decompress(C)[:4])
        assert np.array_equal(cmap.cpu().numpy(), emap)
        assert np.array_equal(x, exp.xadj.astype(np.int64)) and np.array_equal(a, exp.adjncy)
        assert np.array_equal(cw, exp.adjwgt) and np.array_equal(vw, exp.vwgt)


def test_sum_of_equal_records_overflows(lp, oracle_mod, synth_mod):
    # two records of one coarse neighbour whose weights exceed 2^31 - 1 together
    edges = [(0, 2), (0, 3), (1, 2)]
    g = synth_mod.from_edges(4, edges, [2 ** 30, 2 ** 30, 5])
    labels = np.array([0, 1, 2, 2], dtype=np.int32)
    with pytest.raises(OverflowError):
        oracle_mod.contract(g, labels)
    G = lp.lp_graph_from_csr(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
    with pytest.raises(lp.LPError):
        lp.lp_contract(G, labels)
