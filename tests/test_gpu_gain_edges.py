"""Gain table at the degrees where its fill and its updates change hands (one
lane up to 16, one wavefront up to 512, a workgroup above, chunks above the
chunking threshold) and at the block counts where rows turn dense or outgrow
the staging in LDS. Integer work against the definition: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DEGREES = [1, 2, 15, 16, 17, 63, 64, 65, 511, 512, 513, 1000, 2049, 9999, 10000, 10001, 12345]


@pytest.fixture(scope="module")
def graph(synth_mod):
    # vertex i is joined to DEGREES[i] vertices of a common pool, at a stride of its own
    m = max(DEGREES)
    edges = []
    for i, d in enumerate(DEGREES):
        step = [1, 7, 11, 13][i % 4]
        edges += [(i, len(DEGREES) + (j * step) % 12347) for j in range(d)]
    w = [1 + (i * 7919) % 1000 for i in range(len(edges))]
    return synth_mod.from_edges(len(DEGREES) + max(m, 12347), edges, w)


@pytest.mark.parametrize("fmt", ["gap", "plain", "intervals"])
@pytest.mark.parametrize("k", [1, 2, 31, 33, 64, 1023, 1024, 1025])
def test_degree_and_block_edges(lp, oracle_mod, graph, k, fmt):
    g = graph
    if fmt == "plain":
        G = lp.lp_graph_from_csr(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
    else:
        G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, intervals=fmt == "intervals")
    blocks = (np.arange(g.n, dtype=np.int64) * 31 // 40 % k).astype(np.int32)
    rows = np.concatenate([np.arange(len(DEGREES) + 40), np.arange(g.n - 40, g.n)])
    us, bs = np.repeat(rows, k).astype(np.int32), np.tile(np.arange(k), len(rows)).astype(np.int32)
    T = lp.GainTable(G, blocks, k)
    for it in range(3):
        got = T.affinity(us, bs).cpu().numpy().reshape(len(rows), k)
        deg = np.diff(g.xadj.astype(np.int64))
        src = np.repeat(np.arange(g.n), deg)
        sel = np.isin(src, rows)
        A = np.zeros((g.n, k), dtype=np.int64)
        np.add.at(A, (src[sel], blocks[g.adjncy[sel]]), g.adjwgt[sel])
        assert np.array_equal(got, A[rows])
        mv = np.concatenate([np.arange(len(DEGREES)), np.arange(len(DEGREES) + it, g.n, 97)]).astype(np.int32)
        to = ((blocks[mv].astype(np.int64) + 1 + it) % k).astype(np.int32)
        T.move(mv, to)
        blocks[mv] = to
    assert T.info()[2] == 0  # no update missed its entry
    T.free()
