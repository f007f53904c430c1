"""uint8 rows of every length class against the oracle: pool rows are padded to
whole 64-byte matrix-core steps, rows of up to 128 bytes keep their candidate
tiles in registers and longer ones go a step at a time; scratch capacities
above 64; distances above 2^24, which fp32 rounds."""
import numpy as np
import pytest

from helpers import check_graph_invariants
from oracle.oracle import Oracle
from parity import compare_search, compare_states, say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu

N, B = 1_500, 300
# (dim, R, L, P, c, alpha, levels)
CASES = [(1, 8, 32, 64, 2, 1.2, 256), (17, 16, 40, 64, 2, 1.2, 256), (64, 24, 64, 100, 2, 1.2, 256),
         (65, 24, 128, 64, 3, 1.2, 256), (100, 32, 64, 64, 2, 1.2, 256), (127, 64, 128, 128, 1, 1.1, 256),
         (129, 16, 32, 64, 2, 1.2, 256), (200, 48, 128, 64, 4, 1.2, 256), (784, 32, 64, 32, 2, 1.2, 256),
         (2050, 16, 32, 64, 5, 1.2, 256), (200, 24, 64, 64, 2, 1.25, 2), (20, 24, 64, 100, 2, 1.0, 2)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}_r{c[1]}_p{c[3]}_{c[6]}")
def test_u8_rows_match_oracle(case):
    from paper_2608_21163_amd import GrandIndex

    dim, R, L, P, c, alpha, levels = case
    say(f"[u8 rows] {case}")
    cfg = IndexConfig("vamana", "u8", "l2", dim, N + B, R, L, alpha=alpha, P=P, c=c)
    g0 = np.random.default_rng(23)
    x = (g0.integers(0, levels, size=(N + B, dim)) * (255 // (levels - 1))).astype(np.uint8)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=N)
    ids = np.arange(N + B, dtype=np.uint32)

    def same(tag):
        gst = g.export()
        check_graph_invariants(gst, R)
        assert compare_states(gst, o.export(), "vamana") == 0
        say(f"  {tag}: the same lists")

    for s in range(0, N, B):
        assert o.insert(ids[s:s + B], x[s:s + B]) == 0
        g.insert(ids[s:s + B], x[s:s + B])
        same(f"insert {s}")
    assert o.delete(ids[:B]) == 0
    g.delete(ids[:B])
    same("delete")
    st = o.export()
    g.import_graph(x, st["adj"], st["deg"], st["active"], st["medoid"])
    assert o.insert(ids[N:], x[N:]) == 0
    g.insert(ids[N:], x[N:])
    same("insert after import")
    for search in (g.search, g.search_static):
        gi, gd = search(x[:40], 10, 40)
        oi, od = o.search(x[:40], 10, 40)
        assert compare_search(gi, gd, oi, od, 0.0) == 0
