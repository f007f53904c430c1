"""Rows from host memory (copied as blocks and spread to their padded places on
the device) against the same rows in device memory, for rows with and without
padding, through every entry point that takes rows; and an import of more
rows than one block holds."""
import numpy as np
import pytest

from parity import say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu


def _points(dtype, n, d):
    g = np.random.default_rng(5)
    return g.integers(0, 256, (n, d), np.uint8) if dtype == "u8" else g.standard_normal((n, d)).astype(np.float32)


@pytest.mark.parametrize("dtype,metric,dim", [("f32", "l2", 30), ("f32", "l2", 32), ("u8", "l2", 100),
                                              ("u8", "l2", 128), ("f32", "mips", 31)])
def test_host_and_device_rows_agree(dtype, metric, dim):
    import torch

    from paper_2608_21163_amd import GrandIndex
    from paper_2608_21163_amd.grand import STATIC_SCRATCH_BYTES, Reader

    say(f"[host rows] {dtype} {metric} d{dim}")
    n, nq = 900, 77
    cfg = IndexConfig("vamana", dtype, metric, dim, n, 16, 32, mips_norm=50.0 if metric == "mips" else 0.0)
    x, q = _points(dtype, n, dim), _points(dtype, n + nq, dim)[n:]
    ids = np.arange(n, dtype=np.uint32)
    got = []
    for dev in (False, True):
        def put(a):
            return torch.from_numpy(a.view(np.int32) if a.dtype == np.uint32 else a).cuda() if dev else a
        g = GrandIndex.from_config(cfg, max_batch=300)
        for s in range(0, n, 300):
            g.insert(put(ids[s:s + 300]), put(x[s:s + 300]))
        st = g.export()
        g.import_graph(put(x), st["adj"], st["deg"], st["active"], st["medoid"])
        r = Reader(g)
        out = [st["adj"], *g.search(put(q), 10, 32), *g.search_static(put(q), 10, 32), *r.search(put(q), 10, 32)]
        row, stride = dim * x.itemsize, (dim * x.itemsize + 4 * (metric == "mips") + 15) // 16 * 16
        if stride != row:
            # as many results as fit, which leaves no room to stage the packed rows beside them
            m = (STATIC_SCRATCH_BYTES - 3 * 256) // (stride + 2 * 256 * 4)
            used = (m * stride + 255) // 256 * 256 + 2 * (m * 256 * 4)
            assert used <= STATIC_SCRATCH_BYTES < used + m * row
            big = np.tile(q, (m // nq + 1, 1))[:m]
            out += list(g.search_static(put(big), 256, 256))
            assert all(np.array_equal(a, b) for a, b in zip(out[-2:], g.search(put(big), 256, 256)))
        got.append([np.array(a) for a in out])
        r.close()
        g.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_import_of_several_blocks():
    from paper_2608_21163_amd import GrandIndex

    n, d, R = 150_000, 30, 4                                   # 18 MB of packed rows in 128-byte places
    say(f"[host rows] import of {n} x {d}")
    x = _points("f32", n, d)
    adj = ((np.arange(n)[:, None] + np.array([37_501, 61_003, 90_001, 120_011])) % n).astype(np.uint32)
    g = GrandIndex.from_config(IndexConfig("vamana", "f32", "l2", d, n, R, 64), max_batch=64)
    g.import_graph(x, adj, np.full(n, R, np.uint32), np.ones(n, np.uint8), 149_999)
    q = x[:50] + 0.5
    gi, gd = g.search(q, 256, 256)
    assert gi.max() > 140_000 and gi.min() < 40_000
    want = ((x[gi].astype(np.float64) - q[:, None].astype(np.float64)) ** 2).sum(-1)
    assert np.allclose(gd, want, rtol=1e-6, atol=0.0)


@pytest.mark.parametrize("dtype,dim", [("u8", 128), ("u8", 100), ("f32", 32), ("f32", 30)])
def test_results_where_they_lie(dtype, dim):
    """Device buffers of every alignment, and results that overlap another
    buffer of the call, against host buffers (the staged path)."""
    import torch

    from paper_2608_21163_amd import GrandIndex
    from paper_2608_21163_amd.grand import Reader

    say(f"[device results] {dtype} d{dim}")
    n, nq, k = 600, 40, 10
    x, q = _points(dtype, n, dim), _points(dtype, n + nq, dim)[n:]
    g = GrandIndex.from_config(IndexConfig("vamana", dtype, "l2", dim, n, 16, 32), max_batch=n)
    g.insert(np.arange(n, dtype=np.uint32), x)
    want = g.search(q, k, 32)
    r = Reader(g)
    flat = torch.zeros(nq * dim + 64, dtype=torch.uint8 if dtype == "u8" else torch.float32, device="cuda")
    for search in (g.search, r.search):
        for shift in (0, 1, 3, 4, 16):
            dq = flat[shift:shift + nq * dim].view(nq, dim)
            dq.copy_(torch.from_numpy(q))
            ids = torch.full((nq * k + 8,), -1, dtype=torch.int32, device="cuda")
            d = torch.full((nq * k + 8,), -1.0, device="cuda")
            search(dq, k, 32, out_ids=ids[shift % 5:shift % 5 + nq * k].view(nq, k),
                   out_dists=d[shift % 7:shift % 7 + nq * k].view(nq, k))
            assert np.array_equal(ids[shift % 5:shift % 5 + nq * k].cpu().numpy().view(np.uint32).reshape(nq, k), want[0])
            assert np.array_equal(d[shift % 7:shift % 7 + nq * k].cpu().numpy().reshape(nq, k), want[1])
            assert (ids[shift % 5 + nq * k:] == -1).all() and (d[shift % 7 + nq * k:] == -1).all()
        # ids over the queries themselves, distances beside them
        buf = torch.zeros(nq * max(dim, 4 * k) * 4, dtype=torch.uint8, device="cuda")
        dq = buf[:nq * dim * q.itemsize].view(flat.dtype).view(nq, dim)
        dq.copy_(torch.from_numpy(q))
        ids = buf[:nq * k * 4].view(torch.int32).view(nq, k)
        d = torch.zeros(nq, k, device="cuda")
        search(dq, k, 32, out_ids=ids, out_dists=d)
        assert np.array_equal(ids.cpu().numpy().view(np.uint32), want[0])
        assert np.array_equal(d.cpu().numpy(), want[1])
    r.close()
    g.close()
