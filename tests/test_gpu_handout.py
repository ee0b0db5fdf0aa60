"""Tiles handed out in first shares by number and then from counters: lists
that the first shares cover, about cover, and that need counters of every
eighth. Integer work against the oracle: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,half", [(70, 16), (3000, 12), (129000, 16), (131500, 16), (420000, 16), (600000, 20)])
def test_tile_lists(lp, oracle_mod, synth_mod, n, half):
    # circulant graphs: every vertex has 2 * half neighbours, all in small tiles
    off = np.unique(np.concatenate([np.arange(1, half // 2 + 1), 7 * np.arange(half, 2 * half) % (n // 2 - 1) + 1]))[:half]
    nb = np.sort(np.concatenate([(np.arange(n)[:, None] + off) % n, (np.arange(n)[:, None] - off) % n], 1), axis=1)
    d = nb.shape[1]
    g = synth_mod.Graph(n, np.arange(n + 1, dtype=np.uint64) * np.uint64(d), nb.astype(np.int32).ravel())
    exp, _ = oracle_mod.lp_cluster(g, 24, 2, 3)
    for make in (lp.lp_compress, lp.lp_graph_from_csr):
        G = make(g.n, g.xadj.view(np.int64), g.adjncy)
        for config in (None, dict(overlap=1)):
            assert np.array_equal(lp.lp_cluster(G, 24, 2, 3, config=config).cpu().numpy(), exp)
        assert lp.lp_edge_cut(G, exp) == oracle_mod.edge_cut(g, exp)
