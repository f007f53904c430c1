"""The fp32 prune (matrix-core products with an exact repeat of the tests that
their error bound leaves open) against the oracle at the edges of its ranges:
rows shorter and longer than a 32-dimension step, few and many candidates (one
panel of 80, several panels, up to 64 + 128 of a rebuild and 256 of a forward
prune), grids on which alpha * Dist = D holds for many pairs, repeated points,
and values whose products leave the range of the 16-bit pieces."""
import numpy as np
import pytest

from helpers import check_graph_invariants
from oracle.oracle import Oracle
from parity import compare_states, say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu

N, B = 1_500, 300


def _grid(d, levels):
    return lambda g, n: g.integers(0, levels, size=(n, d)).astype(np.float32)


def _normal(d, scale=1.0, offset=0.0):
    return lambda g, n: (offset + scale * g.standard_normal((n, d))).astype(np.float32)


# name: (dim, R, L, P, alpha, points)
CASES = {
    "d1": (1, 16, 32, 64, 1.2, _normal(1)),
    "d33_few": (33, 6, 16, 8, 1.2, _normal(33)),
    "d31_panel_edge": (31, 16, 40, 64, 1.2, _normal(31)),          # at most 80 candidates of a rebuild
    "d100_two_panels": (100, 24, 128, 64, 1.2, _normal(100)),
    "d64_r64_p128": (64, 64, 128, 128, 1.1, _normal(64)),
    "d1000": (1000, 32, 64, 64, 1.2, _normal(1000)),
    "d20_alpha0": (20, 16, 40, 64, 0.0, _normal(20)),
    "d40_offset": (40, 32, 64, 64, 1.2, _normal(40, 1.0, 300.0)),
    "grid_alpha1": (6, 24, 64, 64, 1.0, _grid(6, 3)),               # ties and repeated points
    "grid_alpha125": (12, 32, 128, 100, 1.25, _grid(12, 3)),
    "huge": (16, 24, 64, 64, 1.2, _normal(16, 3e18)),               # distances beyond fp32
    "tiny": (16, 24, 64, 64, 1.2, _normal(16, 1e-15)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_prune_matches_oracle(case):
    from paper_2608_21163_amd import GrandIndex

    say(f"[prune f32] {case}")
    dim, R, L, P, alpha, points = CASES[case]
    cfg = IndexConfig("vamana", "f32", "l2", dim, N + B, R, L, alpha=alpha, P=P)
    x = points(np.random.default_rng(17), N + B)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=N)
    ids = np.arange(N + B, dtype=np.uint32)

    def same(tag):
        gst, ost = g.export(), o.export()
        check_graph_invariants(gst, R)
        # no list may differ: a test that the products leave open is repeated in
        # fp64, and the D of lists and records are the oracle's own (the search's
        # D round apart from them for one distance in some 10^7)
        assert compare_states(gst, ost, "vamana") == 0
        say(f"  {tag}: the same lists")

    for s in range(0, N, B):
        assert o.insert(ids[s:s + B], x[s:s + B]) == 0
        g.insert(ids[s:s + B], x[s:s + B])
        same(f"insert {s}")
    assert o.delete(ids[:B]) == 0
    g.delete(ids[:B])
    same("delete")
    # resumed from an exported state: the stored list distances are recomputed
    st = o.export()
    g.import_graph(x, st["adj"], st["deg"], st["active"], st["medoid"])
    assert o.insert(ids[N:], x[N:]) == 0
    g.insert(ids[N:], x[N:])
    same("insert after import")
