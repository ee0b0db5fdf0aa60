"""Memory kept from freed handles does not starve the caller's allocator: when
that is out of memory, the library gives its own back to the device and asks
again."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_kept_handles_are_given_back(lp, oracle_mod, synth_mod):
    import torch

    g = synth_mod.rmat_scale(12, 8, seed=5)
    exp, _ = oracle_mod.lp_cluster(g, 40, 3, 2)
    G = lp.lp_compress(g.n, g.xadj.view(np.int64), g.adjncy)
    lp.lp_trim_memory()
    C = torch._C
    asked = []

    def alloc(nbytes, stream, ctx):
        full = lp.memory_info()["cached"] > 0  # this allocator's memory: what the library has not kept
        asked.append(full)
        return None if full else C._cuda_cudaCachingAllocator_raw_alloc(int(nbytes), int(stream or 0))

    a = lp.lp_allocator(lp._ALLOC_FN(alloc),
                        lp._FREE_FN(lambda p, stream, ctx: C._cuda_cudaCachingAllocator_raw_delete(int(p))), None)
    lib = lp._load()
    assert lib.lp_set_allocator(ctypes.byref(a)) == lp.LP_OK
    try:
        H = lp.lp_graph_from_csr(g.n, g.xadj.view(np.int64), g.adjncy)
        H.free()
        assert lp.memory_info()["cached"] > 0
        asked.clear()
        lab = lp.lp_cluster(G, 40, 3, 2).cpu().numpy()
        assert asked[0] and not any(asked[1:])  # refused once, then served
        assert lp.memory_info()["cached"] == 0
    finally:
        torch.cuda.synchronize()
        assert lib.lp_set_allocator(None) == lp.LP_OK
    assert np.array_equal(lab, exp)
    G.free()
