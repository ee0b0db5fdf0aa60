"""Buffers of freed handles are kept for later ones: a handle made in memory
that held another graph must be right, whatever the sizes, and emptying the
library's memory gives the kept blocks back."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(lp, g, intervals=False, compressed=True):
    make = (lambda *a: lp.lp_compress(*a, intervals=intervals)) if compressed else lp.lp_graph_from_csr
    G = make(g.n, g.xadj.view(np.int64), g.adjncy, g.adjwgt, g.vwgt)
    lab = lp.lp_cluster(G, 50, 2, 3, config=dict(t_tile=64, t_block=64)).cpu().numpy()  # a plan for one call
    lab0 = lp.lp_cluster(G, 50, 2, 3).cpu().numpy()
    x, a, w, v = (t.cpu().numpy() for t in lp.lp_decompress(G))
    assert np.array_equal(x.view(np.uint64), g.xadj) and np.array_equal(a, g.adjncy)
    if g.adjwgt is not None:
        assert np.array_equal(w, g.adjwgt) and np.array_equal(v, g.vwgt)
    G.free()
    return lab, lab0


def test_reused_buffers(lp, oracle_mod, synth_mod):
    gs = [synth_mod.rmat_scale(s, 8, seed=s) for s in (9, 12, 10, 11)]
    w = synth_mod.rmat_scale(11, 6, seed=7)
    w.adjwgt, w.vwgt = synth_mod.edge_weights(w, 1, 9, 7), synth_mod.vertex_weights(w.n, 1, 3, 7)
    gs.append(w)
    exp = [oracle_mod.lp_cluster(g, 50, 2, 3)[0] for g in gs]
    for it in range(3):
        for g, e in zip(gs, exp):
            for compressed, itv in ((True, False), (True, True), (False, False)):
                for lab in _check(lp, g, itv, compressed):
                    assert np.array_equal(lab, e), it
        if it == 1:
            lp.lp_trim_memory()
            assert lp.memory_info()["cached"] == 0


def test_reused_buffers_in_threads(lp, oracle_mod, synth_mod):
    import torch

    gs = [synth_mod.rmat_scale(10 + k % 3, 8, seed=20 + k) for k in range(4)]
    exp = [oracle_mod.lp_cluster(g, 50, 2, 3)[0] for g in gs]
    bad = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(6):
                    for lab in _check(lp, gs[k]):
                        if not np.array_equal(lab, exp[k]):
                            bad.append(k)
        except Exception as e:  # reported by the assertion below
            bad.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
