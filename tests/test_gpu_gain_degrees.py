"""Gain table where a neighbourhood goes to a wavefront or to a workgroup by its
degree against the others': long ones among many short ones (the limit is 512),
and graphs whose neighbourhoods are all long (twice their mean), with chunked
ones on both sides. Integer work against the definition: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _skewed():
    """Vertices of degree 511 .. 10001 over a ring of 15000 vertices of degree 18 and more."""
    n, special = 15000, [511, 512, 513, 1000, 2049, 4001, 9999, 10001]
    edges = [(i, (i + s) % n) for i in range(n) for s in range(1, 10)]
    step = [7, 11, 13, 17, 19, 23, 29, 31]  # coprime to n: as many distinct neighbours
    edges += [(n + j, v * step[j] % n) for j, d in enumerate(special) for v in range(d)]
    return n + len(special), edges


def _uniform(n, half, special):
    """A circulant of degree 2 * half and a few vertices of other degrees."""
    edges = [(i, (i + s) % n) for i in range(n) for s in range(1, half + 1)]
    edges += [(n + j, v) for j, d in enumerate(special) for v in range(d)]
    return n + len(special), edges


GRAPHS = {"skewed": _skewed, "all-700": lambda: _uniform(1500, 350, [17, 512, 513, 1390, 1450]),
          "all-4100": lambda: _uniform(4400, 2050, [100, 600, 4400])}


@pytest.fixture(scope="module", params=list(GRAPHS))
def graph(request, synth_mod):
    n, edges = GRAPHS[request.param]()
    e = np.unique(np.sort(np.array(edges, dtype=np.int64), axis=1), axis=0)
    src, dst = np.concatenate([e[:, 0], e[:, 1]]), np.concatenate([e[:, 1], e[:, 0]])
    o = np.lexsort((dst, src))
    xadj = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.uint64)
    w = np.tile(1 + np.arange(len(e)) * 7919 % 500, 2)[o].astype(np.int32)
    return synth_mod.Graph(n, xadj, dst[o].astype(np.int32), w)


@pytest.mark.parametrize("fmt", ["gap", "plain", "intervals"])
@pytest.mark.parametrize("k", [3, 1025])
def test_affinities(lp, graph, k, fmt):
    g = graph
    if fmt == "plain":
        G = lp.lp_graph_from_csr(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt)
    else:
        G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, intervals=fmt == "intervals")
    blocks = (np.arange(g.n, dtype=np.int64) * 31 // 40 % k).astype(np.int32)
    rows = np.concatenate([np.arange(60), np.arange(g.n - 40, g.n)])
    us, bs = np.repeat(rows, k).astype(np.int32), np.tile(np.arange(k), len(rows)).astype(np.int32)
    src = np.repeat(np.arange(g.n), np.diff(g.xadj.astype(np.int64)))
    sel = np.isin(src, rows)
    T = lp.GainTable(G, blocks, k)
    for it in range(2):
        A = np.zeros((g.n, k), dtype=np.int64)
        np.add.at(A, (src[sel], blocks[g.adjncy[sel]]), g.adjwgt[sel])
        assert np.array_equal(T.affinity(us, bs).cpu().numpy().reshape(len(rows), k), A[rows])
        mv = np.unique(np.concatenate([np.arange(it, g.n, 53), np.arange(g.n - 8, g.n)])).astype(np.int32)
        to = ((blocks[mv].astype(np.int64) + 1 + it) % k).astype(np.int32)
        T.move(mv, to)
        blocks[mv] = to
    assert T.info()[2] == 0
    T.free()
    G.free()
