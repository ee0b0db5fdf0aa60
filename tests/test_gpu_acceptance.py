"""Acceptance of a round at the edges of its tiles: as many vertices and
proposals as a tile, one more, one less, several tiles, one target for all
proposals (a segment over every tile), a target each, gains of one value (sort
passes left out) and of many. Integer work against the oracle: tolerance 0."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _same(lp, oracle_mod, g, cap, rounds, seed, **config):
    exp, st = oracle_mod.lp_cluster(g, cap, rounds, seed, config.get("subrounds", 1))
    for make in (lp.lp_compress, lp.lp_graph_from_csr):
        G = make(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, g.vwgt)
        lab, gst = lp.lp_cluster(G, cap, rounds, seed, config=config or None, stats=True)
        assert np.array_equal(lab.cpu().numpy(), exp)
        k = gst.rounds_run
        assert gst.proposals == list(st.proposals[:k]) and gst.moves == list(st.moves[:k])


SIZES = [255, 256, 257, 2047, 2048, 2049, 4096, 4097, 8192, 8193, 16383, 16384, 16385, 40000]


@pytest.mark.parametrize("n", SIZES)
def test_one_target_for_all(lp, oracle_mod, synth_mod, n):
    # a star: in the first round every leaf proposes the centre
    g = synth_mod.from_edges(n, [(0, v) for v in range(1, n)])
    _same(lp, oracle_mod, g, max(2, n // 3), 2, 1)
    g.vwgt = synth_mod.vertex_weights(n, 1, 9, 3)
    _same(lp, oracle_mod, g, 2 * n, 2, 1)


@pytest.mark.parametrize("n", SIZES)
def test_a_target_each(lp, oracle_mod, synth_mod, n):
    # a matching with weights 1 .. 2^30: every vertex proposes its partner
    e = [(2 * i, 2 * i + 1) for i in range(n // 2)]
    g = synth_mod.from_edges(n, e, [1 + (i * 2654435761) % (1 << 30) for i in range(len(e))])
    _same(lp, oracle_mod, g, 2, 2, 7)
    _same(lp, oracle_mod, g, 2, 2, 7, subrounds=3)


@pytest.mark.parametrize("n,ef", [(300000, 4), (1100000, 3)])
def test_many_tiles(lp, oracle_mod, synth_mod, n, ef):
    scale = int(np.ceil(np.log2(n)))
    g = synth_mod.rmat(scale, ef * n, seed=11, n_limit=n)
    _same(lp, oracle_mod, g, 64, 3, 5)


@pytest.mark.parametrize("k", [2, 64, 2048, 2049])
def test_refinement_block_weights(lp, oracle_mod, synth_mod, k):
    # blocks left by many vertices at once: summed per workgroup up to 2048 blocks
    g = synth_mod.rmat_scale(14, 8, seed=4)
    g.vwgt = synth_mod.vertex_weights(g.n, 1, 5, 6)
    blocks = ((np.arange(g.n, dtype=np.int64) * 7919) % k).astype(np.int32)
    cap = int(g.vwgt.sum()) // k * 2 + 5
    exp = oracle_mod.lp_refine(g, blocks, k, cap, 4, 9)[0]
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy, None, g.vwgt)
    got = lp.lp_refine(G, blocks, k, cap, 4, 9)
    assert np.array_equal(got.cpu().numpy(), exp)
