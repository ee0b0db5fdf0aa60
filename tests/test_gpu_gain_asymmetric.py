"""Gain table on a graph whose adjacency is not symmetric (which is not checked):
moving a vertex that lists neighbours without a neighbourhood of their own
counts their missing entries and leaves every other affinity right."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CORE, LONE = [3, 40, 300], [5, 60, 400]  # moved by a lane, a wavefront, a workgroup


@pytest.mark.parametrize("fmt", ["gap", "plain", "intervals"])
@pytest.mark.parametrize("k", [2, 5000])
def test_neighbours_without_slots(lp, k, fmt):
    pool, lone = 330, 400
    n = 3 + pool + lone
    if k > n:  # hash slices need more blocks than slots, and blocks are at most the vertices
        n = k
    first_lone = n - lone
    adj = [[] for _ in range(n)]
    for i in range(3):
        for j in range(CORE[i]):
            v = 3 + (7 * j + i) % pool
            adj[i].append(v)
            adj[v].append(i)
        adj[i] += [first_lone + j * (lone // LONE[i]) for j in range(LONE[i])]
    adj = [sorted(a) for a in adj]
    assert [len(adj[i]) for i in range(3)] == [8, 100, 700]
    xadj = np.concatenate([[0], np.cumsum([len(a) for a in adj])]).astype(np.int64)
    flat = np.array([v for a in adj for v in a], dtype=np.int32)
    src = np.repeat(np.arange(n), np.diff(xadj))
    G = (lp.lp_graph_from_csr(n, xadj, flat) if fmt == "plain" else
         lp.lp_compress(n, xadj, flat, intervals=fmt == "intervals"))
    blocks = (np.arange(n) * 13 % k).astype(np.int32)
    T = lp.GainTable(G, blocks, k)
    missing = 0
    for it in range(2):
        mv = np.arange(3, dtype=np.int32)
        to = ((blocks[:3] + 1 + it) % k).astype(np.int32)
        T.move(mv, to)
        missing += sum(LONE[i] for i in range(3) if to[i] != blocks[i])
        blocks[:3] = to
        us = np.concatenate([src, np.arange(first_lone, n)]).astype(np.int32)
        bs = np.concatenate([blocks[flat], blocks[:1].repeat(lone)]).astype(np.int32)
        pairs, cnt = np.unique(src.astype(np.int64) * k + blocks[flat], return_counts=True)
        q = us.astype(np.int64) * k + bs
        at = np.minimum(np.searchsorted(pairs, q), len(pairs) - 1)
        assert np.array_equal(T.affinity(us, bs).cpu().numpy(), np.where(pairs[at] == q, cnt[at], 0)), it
    assert T.info()[2] == missing
    T.free()
    G.free()
