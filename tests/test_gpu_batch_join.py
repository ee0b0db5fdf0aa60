"""Unions of graphs whose arrays are shorter than, or end inside, the sixteen
bytes that one thread joins. Against every graph alone: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("fmt", ["gap", "intervals", "plain"])
def test_join_of_tiny_graphs(lp, oracle_mod, synth_mod, fmt, weighted):
    gs = []
    for i in range(90):
        g = synth_mod.from_edges(1 + i % 3, []) if i % 7 == 3 else synth_mod.random_small(2 + i % 11, 0.6, seed=i)
        if i == 50:
            g = synth_mod.rmat_scale(11, 8, seed=4)
        if weighted:
            if g.two_m == 0:
                continue  # a graph without edges has no weights: not one representation with the others
            g.adjwgt = synth_mod.edge_weights(g, 1, 3000, i)
        gs.append(g)
    if fmt == "plain":
        hs = [lp.lp_graph_from_csr(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt) for g in gs]
    else:
        hs = [lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, intervals=fmt == "intervals") for g in gs]
    outs = lp.lp_batch_cluster(hs, [4] * len(gs), 3, list(range(len(gs))))
    for i, g in enumerate(gs):
        assert np.array_equal(outs[i].cpu().numpy(), oracle_mod.lp_cluster(g, 4, 3, i)[0]), i
    # every edge of the union is cut by singleton labels
    b = lp.lp_batch_create(hs)
    total = sum(int(g.adjwgt.astype(np.int64).sum()) if weighted else g.two_m for g in gs) // 2
    assert lp.lp_edge_cut(b, np.arange(b.n, dtype=np.int32)) == total
