"""Codec calls on more stretches of work than one launch may hold (2^32
threads): records of 2^30 and more neighbours, checked byte by byte against the
format's definition, first-edge IDs of six VarInt bytes among them."""
import numpy as np
import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]

CHUNK = 1000


def _varint(x):
    out = []
    while x >= 0x80:
        out.append((x & 0x7F) | 0x80)
        x >>= 7
    return out + [x]


def _graph(torch, hubs):
    """`hubs` vertices whose only neighbour is the next one, 2^30 and a few more
    times each, then an isolated vertex and one with three neighbours."""
    n = hubs + 2
    deg = [(1 << 30) + 777 * u for u in range(hubs)] + [0, 3]
    xadj = np.concatenate([[0], np.cumsum(np.array(deg, np.int64))])
    adj = torch.empty(int(xadj[-1]), dtype=torch.int32, device="cuda")
    for u in range(hubs):
        adj[xadj[u]:xadj[u + 1]] = (u + 1) % hubs
    adj[xadj[hubs]:] = torch.tensor([0, 1, 5], dtype=torch.int32)
    return n, xadj, adj


def _need(torch, lp, gib):
    lp.lp_trim_memory()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib << 30:
        pytest.skip(f"needs {gib} GiB of free device memory")


def _check_records(torch, G, hubs, xadj, intervals):
    """Offsets and bytes of every record."""
    import paper_2410_19119_amd as m
    offs, data = m.lp_graph_export(G)
    offs = offs.cpu().numpy()
    at = 0
    per = CHUNK + 1 if intervals else CHUNK  # bytes of a whole chunk: the interval count first
    for u in range(hubs):
        assert offs[u] == at, u
        d = int(xadj[u + 1] - xadj[u])
        hdr, nch = _varint(int(xadj[u])), -(-d // CHUNK)
        assert data[at:at + len(hdr)].tolist() == hdr, u
        at += len(hdr)
        table = data[at:at + 4 * (nch - 1)].view(torch.uint8).reshape(-1, 4).to(torch.int64)
        rel = table[:, 0] + (table[:, 1] << 8) + (table[:, 2] << 16) + (table[:, 3] << 24)
        codes = len(hdr) + 4 * (nch - 1)
        assert torch.equal(rel, codes + per * torch.arange(1, nch, device="cuda")), u
        at += 4 * (nch - 1)
        step = (u + 1) % hubs - u
        zig = 2 * step if step > 0 else -2 * step - 1
        first = 1 if intervals else 0
        k = d // CHUNK
        whole = data[at:at + per * k].reshape(k, per)
        assert bool((whole[:, first] == zig).all()), u
        assert int(whole.max(dim=0).values.to(torch.int64).sum()) == zig, u  # every other byte is 0
        at += per * k
        rest = d - CHUNK * k
        if rest:
            assert data[at:at + rest + first].tolist() == [0] * first + [zig] + [0] * (rest - 1), u
            at += rest + first
    end = _varint(int(xadj[hubs]))
    assert data[at:at + len(end)].tolist() == end and offs[hubs] == at
    at += len(end)
    if intervals:
        assert data[at].item() == 0
        at += 1
    tail = end + ([0] if intervals else []) + [2 * (hubs + 1) - 1, 1, 4]
    assert offs[hubs + 1] == at and data[at:].tolist() == tail
    assert offs[hubs + 2] == at + len(tail) == data.numel()


def test_interval_coding(lp):
    """More than 2^23 stretches of 512 threads."""
    import torch
    _need(torch, lp, 130)
    hubs = 17
    n, xadj, adj = _graph(torch, hubs)
    assert int(xadj[-1]) > 1 << 34
    G = lp.lp_compress(n, xadj, adj, intervals=True)
    del adj
    torch.cuda.empty_cache()
    _check_records(torch, G, hubs, xadj, True)
    G.free()
    lp.lp_trim_memory()


def test_gap_coding_both_ways(lp):
    """More than 2^24 stretches of 256 threads, and first-edge IDs beyond 2^35."""
    import torch
    _need(torch, lp, 200)
    hubs = 33
    n, xadj, adj = _graph(torch, hubs)
    assert int(xadj[hubs]) > 1 << 35
    G = lp.lp_compress(n, xadj, adj)
    del adj
    torch.cuda.empty_cache()
    assert G.two_m == int(xadj[-1])
    _check_records(torch, G, hubs, xadj, False)
    torch.cuda.empty_cache()
    lp.lp_trim_memory()
    x = torch.empty(n + 1, dtype=torch.int64, device="cuda")
    a = torch.empty(G.two_m, dtype=torch.int32, device="cuda")
    assert lp._load().lp_decompress(G.handle, x.data_ptr(), a.data_ptr(), None, None, lp._stream()) == lp.LP_OK
    assert np.array_equal(x.cpu().numpy(), xadj)
    for u in range(hubs):
        part = a[xadj[u]:xadj[u + 1]]
        assert int(part.min()) == int(part.max()) == (u + 1) % hubs, u
    assert a[xadj[hubs]:].tolist() == [0, 1, 5]
    G.free()
    lp.lp_trim_memory()
