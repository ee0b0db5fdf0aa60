"""More than 2^28 vertices of low degree: every one of them is rated, visited
and entered into the gain table (a perfect matching, whose answers are known)."""
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


def test_matching(lp):
    import torch
    lp.lp_trim_memory()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of free device memory")
    n = (1 << 28) + 2054
    ids = torch.arange(n, dtype=torch.int32, device="cuda")
    mate = ids ^ 1
    G = lp.lp_graph_from_csr(n, torch.arange(n + 1, device="cuda"), mate)
    # each vertex of a pair moves to the other's cluster
    lab = lp.lp_cluster(G, 2, 1, 1, config=dict(reorder=2))
    assert torch.equal(lab, mate)
    assert lp.lp_edge_cut(G, ids) == n // 2
    assert lp.lp_edge_cut(G, ids & -2) == 0
    C, mp = lp.lp_contract(G, ids & -2)
    assert C.n == n // 2 and C.two_m == 0 and torch.equal(mp, ids >> 1)
    C.free()
    C, mp = lp.lp_contract(G, torch.where(ids >= n - 2 * (n // 4), ids, ids & -2))
    assert C.two_m == 2 * (n // 4)
    del lab, mp
    C.free()
    # blocks by parity: all of a vertex's weight lies in its mate's block
    for gain_table in (0, 1):
        out = lp.lp_refine(G, ids & 1, 2, n, 1, 1, config=dict(gain_table=gain_table))
        assert torch.equal(out, mate & 1), gain_table
        del out
    T = lp.GainTable(G, ids & 1, 2)
    assert bool((T.affinity(ids, mate & 1) == 1).all())
    assert not bool(T.affinity(ids, ids & 1).any())
    T.free()
    G.free()
    torch.cuda.empty_cache()
    lp.lp_trim_memory()
