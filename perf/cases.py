"""The measured work of this framework: what a program that keeps a dynamic
nearest-neighbour index on one GPU has it do, through the public entry points
of `paper_2608_21163_amd` -- searches, streaming rounds (insert, delete,
search), builds and exports -- over the element types, metrics, dimensions and
batch sizes of the configurations in `workloads` and `tests`.

Kinds of case:
  search  one grand_search (or a reader's, or the allocation-free form) over
          nq queries;
  round   one step of a stream in its steady state: insert n points, delete n
          others, search nq queries (CAGRA: delete first).  The pool holds a
          ring of blocks of n ids, one of them free; each pass fills the free
          block and frees the next one, so a pass can be repeated for ever;
  build   an index from nothing: created, filled (insert batches, or the CAGRA
          construction), exported and closed.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2608_21163_amd import GrandIndex
from paper_2608_21163_amd.grand import Reader
from workloads import IndexConfig

INVALID = 0xFFFFFFFF


def _case(kind, **kw):
    c = dict(kind=kind, algo="vamana", dtype="u8", metric="l2", data="mix", dim=128, n_base=1_000_000, R=64, L=128,
             P=64, c=2, alpha=1.2, refresh=0, graph="built", batch=0, delete="uniform", nq=0, k=10, beam=64,
             via="index", host=False, export=False)
    c.update(kw)
    return c


def listed():
    return [
        # one query at a time against a million byte vectors: the latency an interactive lookup sees
        _case("search", name="search_u8_one", refresh=1, nq=1),
        # a full batch of queries against the same index: the search throughput of the headline workload
        _case("search", name="search_u8_10k", refresh=1, nq=10_000),
        # an index resumed from a checkpoint (grand_import_graph) and served through a reader from host memory
        _case("search", name="search_f32_resumed", dtype="f32", data="unit", dim=96, n_base=50_000, graph="imported",
              nq=1_000, beam=128, via="reader", host=True),
        # wide result lists of text embeddings by inner product: k = 100 at the largest beam
        _case("search", name="search_mips768_k100", dtype="f32", metric="mips", data="ip", dim=768, n_base=100_000,
              nq=1_000, k=100, beam=256),
        # the headline stream: a million 128-d byte vectors, 1% of them replaced per round
        _case("round", name="round_u8_1m", refresh=1, batch=10_000, nq=10_000),
        # a trickle of updates and queries on the same index: launches and passes over the pool count
        _case("round", name="round_u8_trickle", refresh=1, batch=100, nq=100),
        # byte vectors of an odd length (100-d embeddings) at half the degree
        _case("round", name="round_u8_d100", dim=100, n_base=200_000, R=32, batch=2_000, nq=2_000),
        # the sliding window of a million 96-d fp32 image descriptors: the oldest 1% make room
        _case("round", name="round_f32_window", dtype="f32", data="unit", dim=96, delete="oldest", batch=10_000,
              nq=10_000),
        # long fp32 rows (960-d image features)
        _case("round", name="round_f32_d960", dtype="f32", data="relu", dim=960, n_base=100_000, batch=2_000,
              nq=2_000, beam=128),
        # the fixed-degree variant on 100-d word embeddings by inner product
        _case("round", name="round_cagra_ip100", algo="cagra", dtype="f32", metric="ip", data="student", dim=100, L=64,
              batch=10_000, nq=10_000),
        # a small index of a host program, saved after every round
        _case("round", name="round_small_saved", dtype="f32", data="gauss", dim=32, n_base=10_000, R=32, L=64,
              batch=500, nq=100, host=True, export=True),
        # the CAGRA graph of a whole set in one call, and its export
        _case("build", name="build_cagra_100k", algo="cagra", dtype="f32", metric="ip", data="student", dim=100,
              n_base=100_000, L=64, export=True),
    ]


def _log(rng, a, b):
    return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm, odd
    ones among them."""
    kind = rng.choice(["search", "search", "round", "round", "round", "build"])
    algo = "cagra" if rng.random() < 0.25 else "vamana"
    dtype = rng.choice(["u8", "f32"])
    metric, data = "l2", "mix"
    if dtype == "f32":
        data = rng.choice(["unit", "relu", "gauss"])
        if algo == "cagra" and rng.random() < 0.7:
            metric, data = "ip", "student"
        elif rng.random() < 0.25:
            metric, data = "mips", "ip"
    dim = _log(rng, 16, 512) if dtype == "u8" else _log(rng, 16, 1000)
    if rng.random() < 0.4:  # the usual lengths beside the odd ones
        dim = rng.choice([64, 96, 100, 128, 256] if dtype == "u8" else [32, 96, 100, 256, 768, 960])
    most = (50_000_000 if dtype == "u8" else 20_000_000) // dim
    n_base = _log(rng, 4_000, max(8_000, min(500_000, most)))
    R = rng.choice([16, 24, 32, 48, 64])
    L = rng.choice([64, 96, 128])
    graph = "built"
    if kind == "search" and dtype == "f32" and metric != "mips" and rng.random() < 0.5:
        graph, n_base = "imported", min(n_base, 50_000)
    host = rng.random() < 0.3
    if kind == "build":
        n_base = min(n_base, 12_000 if host else 50_000, 8_000_000 // dim)
    k = rng.choice([1, 10, 10, 10, 50, 100])
    beam = rng.choice([b for b in (32, 64, 100, 128, 200, 256) if b >= k])
    batch = _log(rng, 20, max(40, n_base // 50)) if kind == "round" else 0
    nq = 0 if kind == "build" else _log(rng, 1, 10_000 if dim <= 256 else 2_000)
    return _case(kind, algo=algo, dtype=dtype, metric=metric, data=data, dim=dim, n_base=n_base, R=R, L=L,
                 P=rng.choice([32, 64, 64, 100]), c=rng.choice([1, 2, 2, 3]), alpha=rng.choice([1.0, 1.2, 1.2, 1.4]),
                 graph=graph, batch=batch, delete=rng.choice(["uniform", "oldest"]), nq=nq, k=k, beam=beam,
                 via=rng.choice(["index", "index", "reader", "static"]) if nq * dim <= 200_000 and nq * k <= 200_000 else "index",
                 host=host, export=kind == "build")


# ------------------------------------------------------------------- inputs
def _points(case, n, seed):
    """n points on the GPU, from the mixtures of `workloads` (clusters of
    about 2,000 points)."""
    g = torch.Generator(device="cuda").manual_seed(seed * 8 + 1)
    d, data = case["dim"], case["data"]
    nc = max(4, case["n_base"] // 2_000)

    def normal(*s):
        return torch.randn(*s, generator=g, device="cuda")

    if data == "gauss":
        return normal(n, d)
    centres = torch.rand(nc, d, generator=g, device="cuda") * 255 if data == "mix" else normal(nc, d)
    scale = 0.1 + 0.9 * torch.rand(d, generator=g, device="cuda")
    lengths = 0.5 + torch.rand(nc, 1, generator=g, device="cuda")
    if data == "ip":  # cluster centres of different lengths
        centres = centres * lengths
    out = torch.empty(n, d, dtype=torch.uint8 if data == "mix" else torch.float32, device="cuda")
    for s in range(0, n, 65_536):
        m = min(65_536, n - s)
        mu = centres[torch.randint(0, nc, (m,), generator=g, device="cuda")]
        if data == "mix":
            x = (mu + 20.0 * normal(m, d)).round_().clamp_(0, 255)
        elif data == "relu":
            x = torch.relu(scale * (mu + 0.5 * normal(m, d)))
        elif data == "student":  # three degrees of freedom
            x = mu + 0.3 * normal(m, d) / (normal(3, m, d).square().sum(0) / 3.0).sqrt()
            x = x / x.norm(dim=1, keepdim=True)
        elif data == "ip":
            x = mu + 0.35 * normal(m, d)
            x = x * (0.99 * _norm_bound(case) / x.norm(dim=1, keepdim=True)).clamp(max=1.0)
        else:
            x = mu + 0.5 * normal(m, d)
            x = x / x.norm(dim=1, keepdim=True)
        out[s:s + m] = x.to(out.dtype)
    return out


def _norm_bound(case):
    return 1.5 * math.sqrt(case["dim"])


def _ring(case):
    """(ids per block, blocks) of the pool: a round's ring has one free block."""
    n = case["batch"]
    return (n, case["n_base"] // n + 1) if n else (case["n_base"], 1)


def _config(case):
    n, blocks = _ring(case)
    return IndexConfig(case["algo"], case["dtype"], case["metric"], case["dim"], n * blocks, case["R"], case["L"],
                       alpha=case["alpha"], P=case["P"], c=case["c"],
                       mips_norm=_norm_bound(case) if case["metric"] == "mips" else 0.0)


def _build_batch(case):
    return max(256, min(10_000, case["n_base"] // 8))


def _index(case):
    return GrandIndex.from_config(_config(case), max_batch=max(_build_batch(case), case["batch"]),
                                  stream=torch.cuda.current_stream().cuda_stream)


def _fill(case, g, ids, x):
    step = _build_batch(case)
    for s in range(0, len(ids), step):
        g.insert(ids[s:s + step], x[s:s + step])


def _knn_graph(case, x, seed):
    """Lists of R/2 nearest neighbours and R/2 random links of every point, by
    plain torch: the checkpoint that an imported index is resumed from."""
    n, r = len(x), case["R"]
    g = torch.Generator(device="cuda").manual_seed(seed * 8 + 2)
    sq = x.square().sum(1)
    me = torch.arange(n, device="cuda")[:, None]
    near = torch.empty(n, r // 2, dtype=torch.int64, device="cuda")
    for s in range(0, n, 4_096):
        dist = -2.0 * (x[s:s + 4_096] @ x.T)
        if case["metric"] == "l2":
            dist += sq
        dist[torch.arange(len(dist), device="cuda"), torch.arange(s, s + len(dist), device="cuda")] = float("inf")
        near[s:s + 4_096] = dist.topk(r // 2, dim=1, largest=False).indices
    rows = torch.cat([near, torch.randint(0, n, (n, r - r // 2), generator=g, device="cuda")], 1)
    rows = rows.masked_fill(rows == me, INVALID).sort(1).values
    rows[:, 1:] = rows[:, 1:].masked_fill(rows[:, 1:] == rows[:, :-1], INVALID)
    rows = rows.sort(1).values
    return rows, (rows != INVALID).sum(1)


def _queries(case, seed):
    """Fresh draws of the points' own distribution."""
    x = _points(case, case["n_base"] + case["nq"], seed)
    return x[:case["n_base"]], x[case["n_base"]:].clone()


def _out(case):
    shape = (case["nq"], case["k"])
    if case["host"]:
        return np.zeros(shape, np.uint32), np.zeros(shape, np.float32)
    return torch.zeros(shape, dtype=torch.int32, device="cuda"), torch.zeros(shape, device="cuda")


def _hosted(case, x):
    return x.cpu().numpy() if case["host"] else x


def prepare(case, seed):
    s = dict(case=case)
    if case["kind"] == "build":
        x = _points(case, case["n_base"], seed)
        s["x"] = _hosted(case, x)
        s["ids"] = _hosted(case, torch.arange(len(x), dtype=torch.int32, device="cuda"))
        if case["algo"] == "cagra":
            knn = min(128, 2 * case["R"])
            g = torch.Generator(device="cuda").manual_seed(seed * 8 + 3)
            # distinct random positions other than a point's own: offsets, one in each of knn equal ranges
            n, w = len(x), (len(x) - 1) // knn
            off = torch.randint(0, w, (n, knn), generator=g, device="cuda") + torch.arange(knn, device="cuda") * w
            init = (torch.arange(n, device="cuda")[:, None] + 1 + off) % n
            s["init"], s["knn"] = _hosted(case, init.to(torch.int32)), knn
        return s
    n, blocks = _ring(case)
    total = n * blocks
    x, q = _queries(dict(case, n_base=total), seed)
    g = _index(case)
    if case["graph"] == "imported":
        rows, deg = _knn_graph(case, x, seed)
        g.import_graph(x, rows.cpu().numpy().astype(np.uint32), deg.cpu().numpy().astype(np.uint32),
                       np.ones(total, np.uint8), 0)
    else:
        gen = torch.Generator(device="cuda").manual_seed(seed * 8 + 4)
        ids = torch.arange(total, device="cuda") if case["delete"] == "oldest" or not case["batch"] \
            else torch.randperm(total, generator=gen, device="cuda")
        ids = ids.to(torch.int32)
        live = total - case["batch"]
        _fill(case, g, ids[:live], x[:live])
        for _ in range(case["refresh"]):  # every batch again, against the whole set
            step = _build_batch(case)
            for a in range(0, live, step):
                b = min(live, a + step)
                g.delete(ids[a:b])
                g.insert(ids[a:b], x[a:b])
        if case["batch"]:
            s["ids"], s["x"] = _hosted(case, ids), _hosted(case, x)
            s["at"], s["n"], s["blocks"] = 0, n, blocks
    s["index"], s["q"], s["out"] = g, _hosted(case, q), _out(case)
    s["reader"] = Reader(g) if case["via"] == "reader" else None
    torch.cuda.synchronize()
    return s


def _search(s):
    case, (ids, dists) = s["case"], s["out"]
    if case["via"] == "reader":
        search = s["reader"].search
    else:
        search = s["index"].search_static if case["via"] == "static" else s["index"].search
    search(s["q"], case["k"], case["beam"], out_ids=ids, out_dists=dists)
    return ids, dists


def _saved(g):
    st = g.export()
    return [st["adj"], st["deg"], st["active"], st["medoid"]]


def run(s):
    case = s["case"]
    if case["kind"] == "search":
        return _search(s)
    if case["kind"] == "build":
        g = _index(case)
        if case["algo"] == "cagra":
            g.build_cagra(s["ids"], s["x"], s["init"], s["knn"], 6, 16)
        else:
            _fill(case, g, s["ids"], s["x"])
        out = _saved(g)
        g.close()
        return out
    g, n, blocks = s["index"], s["n"], s["blocks"]
    free, nxt = (s["at"] - 1) % blocks, s["at"]  # the free block, and the one that is freed
    s["at"] = (s["at"] + 1) % blocks
    if case["algo"] == "cagra" and case["n_base"] > 2 * n:
        g.delete(s["ids"][nxt * n:(nxt + 1) * n])
        g.insert(s["ids"][free * n:(free + 1) * n], s["x"][free * n:(free + 1) * n])
    else:
        g.insert(s["ids"][free * n:(free + 1) * n], s["x"][free * n:(free + 1) * n])
        g.delete(s["ids"][nxt * n:(nxt + 1) * n])
    out = list(_search(s))
    return out + _saved(g) if case["export"] else out


# ------------------------------------------------- what a pass cannot do without
def work(case):
    """Bytes and operations of one pass.  A search of beam l expands about
    1.05 l nodes (one list each) and needs the rows of about 0.35 R new
    neighbours of each, as the library's counters show on these data; an
    update reads and writes the lists that it changes, about R per point, and
    reads the rows that their prunes need (each row of the pool once); a
    delete batch reads every list once to find the edges into it."""
    esize = 1 if case["dtype"] == "u8" else 4
    d, R, n = case["dim"], case["R"], case["batch"]
    row = d * esize
    N = case["n_base"]

    def search(nq, beam):
        hops = min(N, 1.05 * beam)
        rows = min(N, 0.35 * R * hops)
        # a row or list that several searches of a call need comes from memory once at least
        return nq * row + min(N, nq * hops) * 4 * R + min(N, nq * rows) * row, nq * rows * 2 * d

    b = f = 0.0
    if case["kind"] == "build":
        if case["algo"] == "cagra":
            # per round and point: 4 x 16 candidates joined pairwise, one list read and written
            return {"bytes": 6.0 * N * (row + 3 * 8 * 2 * R), "flops": 6.0 * N * 1500 * 2 * d}
        n, searches = N, 1
    else:
        searches = 2 if n else 0
    if case["kind"] != "search":
        sb, sf = search(n, case["L"])
        if case["algo"] == "cagra":
            b, f = sb + n * R * 4 * (12 + 2 * R), sf
            if searches > 1:
                b += N * R * 4 + n * R * 4 * (2 + 2 * R)
        else:
            lists = min(N, n * R)
            for _ in range(searches):
                b += sb + lists * 8 * R + min(N, 0.5 * lists * 1.2 * R) * row
                f += sf + 0.5 * lists * 0.3 * R * R * 2 * d
            if searches > 1:
                b += N * R * 4 + min(N, n * (50 + 2 * R)) * row
                f += n * 2 * R * 50 * 2 * d
    if case["nq"]:
        sb, sf = search(case["nq"], case["beam"])
        b, f = b + sb + case["nq"] * case["k"] * 8, f + sf
    if case["export"]:
        b += 2.0 * N * R * 4
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Byte vectors: integer distances, ordered with their ids.  fp32: sums of
    64 bits rounded once, so another order of a sum moves a distance by one
    part in 1.7e7 at most and exchanges ids only where two distances tie; a
    list that a tie changes can pass on to a few results of the rounds that
    follow."""
    if case["dtype"] == "u8":
        return "exact"
    if case["kind"] == "search":
        return {"rel": 1e-6, "max": 1e-4, "differ": 1e-3}
    return {"rel": 1e-5, "max": 0.05, "differ": 1e-3}


def exact(case, seed):
    """The searches of imported graphs: the beam search (the l closest keys,
    the smallest unexpanded one expanded next, at most 2 l expansions) in 64
    bits.  A graph that the library builds itself takes minutes here."""
    if case["graph"] != "imported":
        return None
    x, q = _queries(case, seed)
    rows, _ = _knn_graph(case, x, seed)
    n, nq, ell = len(x), case["nq"], case["beam"]
    xd, qd = x.double(), q.double()
    ids = torch.full((nq, ell), INVALID, device="cuda")
    dist = torch.full((nq, ell), float("inf"), dtype=torch.float64, device="cuda")
    done = torch.zeros(nq, ell, dtype=torch.bool, device="cuda")
    every = torch.arange(nq, device="cuda")

    def to(v):  # distances of every query to its ids v
        out = torch.full(v.shape, float("inf"), dtype=torch.float64, device="cuda")
        step = max(1, 30_000_000 // (v.shape[1] * case["dim"]))
        for a in range(0, nq, step):
            y = xd[v[a:a + step].clamp(max=n - 1)]
            z = qd[a:a + step, None]
            out[a:a + step] = (y - z).square().sum(2) if case["metric"] == "l2" else -(y * z).sum(2)
        return out.masked_fill(v == INVALID, float("inf"))

    ids[:, 0] = 0
    dist[:, :1] = to(ids[:, :1])
    for _ in range(2 * ell):
        left = (ids != INVALID) & ~done
        if not bool(left.any()):
            break
        e = left.int().argmax(1)
        some = left.any(1)
        done[every, e] |= some
        new = rows[ids[every, e].clamp(max=n - 1)].masked_fill(~some[:, None], INVALID)
        new = new.masked_fill((new[:, :, None] == ids[:, None, :]).any(2), INVALID)
        ids, dist = torch.cat([ids, new], 1), torch.cat([dist, to(new)], 1)
        done = torch.cat([done, torch.zeros_like(new, dtype=torch.bool)], 1)
        by_id = ids.argsort(1)
        order = by_id.gather(1, dist.gather(1, by_id).argsort(dim=1, stable=True))[:, :ell]
        ids, dist, done = ids.gather(1, order), dist.gather(1, order), done.gather(1, order)
    k = case["k"]
    return [ids[:, :k].cpu().numpy().astype(np.uint32), dist[:, :k].cpu().numpy()]
