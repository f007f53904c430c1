"""The construction's joins and merges at the edges of their ranges against the
oracle, slot for slot: rows shorter and longer than a K step, one to 32 samples
per list (one to eight candidate tiles), lists of up to 128 entries, repeated
points and distances that tie, offsets that cancel, and ranges of nodes whose
proposals exceed the record buffers, so that their blocks are launched again."""
import numpy as np
import pytest

from oracle.oracle import Oracle
from parity import say
from workloads import IndexConfig
from workloads.generators import cagra_init_lists

pytestmark = pytest.mark.gpu


def _normal(d, scale=1.0, offset=0.0):
    return lambda g, n: (offset + scale * g.standard_normal((n, d))).astype(np.float32)


def _grid(d, levels, dtype=np.float32):
    return lambda g, n: g.integers(0, levels, (n, d)).astype(dtype)


# name: (dtype, metric, dim, n, knn, R, sample, rounds, points)
CASES = {
    "ip_d100_k128": ("f32", "ip", 100, 1_500, 128, 64, 16, 4, _normal(100)),
    "ip_d7_s1": ("f32", "ip", 7, 600, 33, 16, 1, 3, _normal(7)),
    "l2_d33_s17": ("f32", "l2", 33, 900, 70, 32, 17, 3, _normal(33)),
    "l2_d1": ("f32", "l2", 1, 500, 16, 8, 8, 2, _normal(1)),
    "l2_offset": ("f32", "l2", 40, 800, 32, 16, 8, 3, _normal(40, 0.01, 100.0)),
    "l2_grid_ties": ("f32", "l2", 5, 900, 64, 24, 16, 3, _grid(5, 3)),
    "u8_d200": ("u8", "l2", 200, 900, 128, 32, 16, 3, _grid(200, 256, np.uint8)),
    "u8_d20_ties": ("u8", "l2", 20, 900, 48, 24, 32, 3, _grid(20, 2, np.uint8)),
    "l2_d8_ranges": ("f32", "l2", 8, 16_000, 64, 32, 16, 3, _normal(8)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_joins_match_oracle(case):
    from paper_2608_21163_amd import GrandIndex

    dtype, metric, dim, n, K, R, S, rounds, points = CASES[case]
    say(f"[join] {case}")
    x = points(np.random.default_rng(31), n)
    cfg = IndexConfig("cagra", dtype, metric, dim, n, R, 64)
    ids = np.random.default_rng(32).permutation(n).astype(np.uint32)
    init = cagra_init_lists(n, K, 33)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=256)
    assert o.build_cagra(ids, x, init, K, rounds, S) == 0, o.last_error()
    g.build_cagra(ids, x, init, K, rounds, S)
    gst, ost = g.export(), o.export()
    diff = np.flatnonzero((gst["adj"] != ost["adj"]).any(1) | (gst["deg"] != ost["deg"]))
    assert diff.size == 0, (diff.size, diff[:5])
    assert gst["medoid"] == ost["medoid"]
    g.close()


RCAP = 20 << 20            # records of the buffers that a round's ranges fill


@pytest.mark.parametrize("dtype,dim,far,clusters,K,R,S", [("f32", 8, 4_800, 320, 64, 32, 32),
                                                          ("u8", 20, 19_200, 2_400, 32, 16, 16)])
def test_ranges_that_exceed_the_record_buffers(dtype, dim, far, clusters, K, R, S):
    """The first `far` points hold initial lists over far clusters, whose joins
    propose nothing; the others hold their own cluster, all of whose pairs are
    proposed.  The first range (sized for every pair of 2 S candidates) covers
    far points only, so the second is sized for no proposals and takes all the
    rest: more than the buffers hold (26.2M and 23.0M proposals)."""
    from paper_2608_21163_amd import GrandIndex

    assert 0.9 * RCAP / (2 * S * (2 * S - 1)) < far - 5
    w = K + 1
    n = far + clusters * w
    g0 = np.random.default_rng(41)
    if dtype == "u8":
        centre = g0.integers(4, 252, (clusters, dim))
        x = np.concatenate([g0.integers(0, 256, (far, dim)), (centre[:, None] + g0.integers(-3, 4, (clusters, w, dim))
                                                              ).reshape(-1, dim)]).astype(np.uint8)
    else:
        centre = 100.0 * g0.standard_normal((clusters, dim))
        x = np.concatenate([100.0 * g0.standard_normal((far, dim)),
                            (centre[:, None] + g0.standard_normal((clusters, w, dim))).reshape(-1, dim)])
        x = x.astype(np.float32)
    init = np.empty((n, K), np.uint32)
    for p in range(far):
        init[p] = far + w * g0.choice(clusters, K, replace=False) + g0.integers(0, w, K)
    mates = np.arange(w)
    others = np.stack([np.delete(mates, m) for m in mates])
    init[far:] = (far + w * np.arange(clusters)[:, None, None] + others[None]).reshape(-1, K)
    say(f"[join ranges] {dtype} d{dim} n {n}")
    cfg = IndexConfig("cagra", dtype, "l2", dim, n, R, 64)
    ids = np.arange(n, dtype=np.uint32)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=256)
    assert o.build_cagra(ids, x, init, K, 1, S) == 0, o.last_error()
    g.set_timing(True)
    g.build_cagra(ids, x, init, K, 1, S)
    # groupings of the samples, of the second range, of the reverse edges, and
    # of at least one launch for the blocks that found no room
    calls = g.stats()["phase_calls"]["group"]
    say(f"  {calls} groupings")
    assert calls >= 4
    gst, ost = g.export(), o.export()
    diff = np.flatnonzero((gst["adj"] != ost["adj"]).any(1) | (gst["deg"] != ost["deg"]))
    assert diff.size == 0, (diff.size, diff[:5])
    assert gst["medoid"] == ost["medoid"]
    g.close()
