"""Grouping of reverse-edge records over pools of every bucket width (64 to
4096 targets per bucket; the edges where the width doubles): inserts and
deletes of points spread over the whole id range, against the oracle."""
import numpy as np
import pytest

from helpers import check_graph_invariants
from oracle.oracle import Oracle
from parity import compare_states, say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [40, 64, 65, 700, 16_384, 16_385, 40_000, 524_288, 1_048_577])
def test_grouping_of_every_bucket_width(cap):
    from paper_2608_21163_amd import GrandIndex

    say(f"[grouping] capacity {cap}")
    n = min(cap, 900)
    g0 = np.random.default_rng(cap)
    ids = np.sort(g0.choice(cap, n, replace=False)).astype(np.uint32)
    ids[0], ids[-1] = 0, cap - 1
    ids = g0.permutation(np.unique(ids)).astype(np.uint32)
    n = len(ids)
    x = g0.integers(0, 256, (n, 32), np.uint8)
    cfg = IndexConfig("vamana", "u8", "l2", 32, cap, 16, 32)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=n)
    h = n // 2
    for a, b in ((0, h), (h, n)):
        assert o.insert(ids[a:b], x[a:b]) == 0
        g.insert(ids[a:b], x[a:b])
    assert o.delete(ids[h // 2:h]) == 0
    g.delete(ids[h // 2:h])
    gst = g.export()
    check_graph_invariants(gst, cfg.R)
    assert compare_states(gst, o.export(), "vamana") == 0
    g.close()
