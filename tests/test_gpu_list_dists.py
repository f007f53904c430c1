"""The distances that rebuilds take from lists and records (fp32): the fp64 sum
in dimension order, rounded once, whichever kernel produced them, so that a
list is a function of the graph and the vectors.

D(u, j) is 1 + 2^-24, half way between two fp32 values, plus terms of 2^-54
that a sum in dimension order loses (it rounds to 1) and that a sum over lanes
keeps (it rounds to 1 + 2^-23).  Dist(i, j) is 1 + 2^-23, so with alpha = 1 a
selected i kills j in u's rebuild only by the second value."""
import numpy as np
import pytest

from helpers import INVALID, canonical_rows, check_graph_invariants, rows_to_adj
from oracle.oracle import Oracle
from parity import compare_states, say
from workloads import IndexConfig

pytestmark = pytest.mark.gpu

U, I, J, K, M, P = range(6)
ULP = np.float32(1.0) + np.float32(2.0 ** -23)


def _points(d, dist):
    x = np.zeros((6, d), np.float32)
    x[J] = 2.0 ** -27
    x[J, 0], x[J, 1] = 1.0, 2.0 ** -12
    x[I, 0] = 0.25
    x[I, 2] = 0.66
    while dist(x[I], x[J]) < ULP:
        x[I, 2] = np.nextafter(x[I, 2], np.float32(1.0))
    x[K, 0], x[M, 3], x[P, 4] = -3.0, -2.9, 0.1
    assert dist(x[U], x[J]) == 1.0 and dist(x[I], x[J]) == ULP and dist(x[U], x[I]) < 1.0
    return x


def _sides(x, R, lists, start, c=2):
    from paper_2608_21163_amd import GrandIndex

    cfg = IndexConfig("vamana", "f32", "l2", x.shape[1], 6, R, 16, alpha=1.0, c=c)
    sides = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=6)
    adj, deg = rows_to_adj([lists.get(v, []) for v in range(6)], R)
    active = np.array([v in lists for v in range(6)], np.uint8)
    for s in sides:
        s.import_graph(x, adj, deg, active, start)
    return sides


def _insert(sides, x, v):
    for s in sides:
        s.insert(np.array([v], np.uint32), x[v:v + 1])


def _same(o, g, want):
    a, b = canonical_rows(g.export()["adj"]), canonical_rows(o.export()["adj"])
    assert set(b[U].tolist()) - {INVALID} == want
    assert np.array_equal(a, b), (a.tolist(), b.tolist())


def _dist(d):
    return Oracle(IndexConfig("vamana", "f32", "l2", d, 6, 2, 16)).dist


DIMS = [8, 33, 96, 200, 400, 600, 1000]


@pytest.mark.parametrize("d", DIMS)
def test_records_of_an_insert(d):
    say(f"[list distances] record of an insert, d{d}")
    x = _points(d, _dist(d))
    o, g = _sides(x, 2, {U: [I, K], I: [U], K: [U]}, U)
    _insert((o, g), x, J)
    _same(o, g, {I, J})
    g.close()


@pytest.mark.parametrize("resumed", [False, True])
@pytest.mark.parametrize("d", DIMS)
def test_list_of_a_new_point(d, resumed):
    say(f"[list distances] list of a new point, d{d}, resumed {resumed}")
    x = _points(d, _dist(d))
    o, g = _sides(x, 2, {J: [K], K: [J]}, K)
    _insert((o, g), x, U)
    _same(o, g, {J, K})
    if resumed:
        st = g.export()
        g.import_graph(x, st["adj"], st["deg"], st["active"], st["medoid"])
    _insert((o, g), x, I)
    _same(o, g, {I, J})
    g.close()


@pytest.mark.parametrize("c", [2, 4, 5])
@pytest.mark.parametrize("d", DIMS)
def test_records_of_a_delete(d, c):
    say(f"[list distances] records of a delete, d{d}, c {c}")
    x = _points(d, _dist(d))
    lists = {U: [P, I, K], P: [U, J, M], I: [P], J: [P], K: [P], M: [P]}
    o, g = _sides(x, 3, lists, U, c)
    for s in (o, g):
        s.delete(np.array([P], np.uint32))
    _same(o, g, {I, J, M})
    g.close()


@pytest.mark.parametrize("dtype,d,R,P", [("f32", 20, 24, 64), ("f32", 300, 16, 100), ("f32", 7, 15, 64),
                                         ("u8", 128, 24, 64), ("u8", 40, 18, 64), ("u8", 200, 64, 128)])
def test_updates_after_an_import(dtype, d, R, P):
    """An import leaves the list distances to the first rebuild that prunes a
    node; lists grow, shrink and are pruned with some of them known."""
    from paper_2608_21163_amd import GrandIndex

    say(f"[list distances] updates after an import, {dtype} d{d} R{R} P{P}")
    n, b = 1_200, 100
    cfg = IndexConfig("vamana", dtype, "l2", d, n, R, 48, P=P)
    g0 = np.random.default_rng(51)
    x = g0.integers(0, 256, (n, d)).astype(np.uint8) if dtype == "u8" else g0.standard_normal((n, d)).astype(np.float32)
    ids = g0.permutation(n).astype(np.uint32)
    o, g = Oracle(cfg), GrandIndex.from_config(cfg, max_batch=400)
    for s in range(0, 800, 400):
        assert o.insert(ids[s:s + 400], x[ids[s:s + 400]]) == 0
    st = o.export()
    g.import_graph(x, st["adj"], st["deg"], st["active"], st["medoid"])
    for k in range(4):
        new, old = ids[800 + k * b:800 + (k + 1) * b], ids[k * b:(k + 1) * b]
        for s in (o, g):
            s.insert(new, x[new])
            s.delete(old)
        gst = g.export()
        check_graph_invariants(gst, R)
        assert compare_states(gst, o.export(), "vamana") == 0
    g.close()
