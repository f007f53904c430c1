"""Searches of rows of every lane layout (8 lanes a row up to 32 chunks of 16
bytes, 16 up to 64, 32 up to 128, 64 up to 256; the longest rows with 16 lanes
where few searches run) against the oracle: both ends of each class, beams of
one, two and four register rows, single queries and more than the SIMDs."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from parity import compare_search, say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu

CASES = [("f32", "l2", d) for d in (32, 33, 128, 129, 131, 256, 257, 300, 512, 513, 700, 1024)] + \
        [("f32", "ip", d) for d in (130, 259, 515, 771)] + [("u8", "l2", d) for d in (513, 1030, 2100, 4096)]


@pytest.mark.parametrize("dtype,metric,dim", CASES)
def test_search_of_every_row_layout(dtype, metric, dim):
    from paper_2608_21163_amd import GrandIndex

    say(f"[search rows] {dtype} {metric} d{dim}")
    n, R = 700, 12
    g0 = np.random.default_rng(dim)
    if dtype == "u8":
        x = g0.integers(0, 256, (n, dim), np.uint8)
    else:
        x = g0.standard_normal((n, dim)).astype(np.float32)
    cfg = IndexConfig("cagra" if metric == "ip" else "vamana", dtype, metric, dim, n, R, 32)
    # a graph of random links: every search expands its whole beam
    adj = ((np.arange(n)[:, None] + 1 + np.stack([g0.choice(n - 1, R, replace=False) for _ in range(n)])) % n)
    adj = adj.astype(np.uint32)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=64)
    for side in (o, g):
        side.import_graph(x, adj, np.full(n, R, np.uint32), np.ones(n, np.uint8), 3)
    for nq, k, beam in ((1, 10, 64), (37, 20, 128), (9, 100, 256), (1_100, 60, 64)):
        q = g0.integers(0, 256, (nq, dim), np.uint8) if dtype == "u8" else \
            g0.standard_normal((nq, dim)).astype(np.float32)
        gi, gd = g.search(q, k, beam)
        oi, od = o.search(q, k, beam)
        compare_search(gi, gd, oi, od, 0.0 if dtype == "u8" else 0.01)
    g.close()
