"""Performance cases: what a program built on this library has it do.

Every case names an operation (``op``), a graph and its partition, the build
options and the number of query pairs:

* ``build``     ``build_index`` on device arrays, then one batch of queries
                (a new road network goes live: the index is built and used);
* ``reweight``  new edge weights on a captured index, then one batch (traffic
                update);
* ``batch``     ``query_batch`` on a resident index, device pairs;
* ``host``      ``query_batch_host``: host pairs in, host answers out;
* ``serve``     a burst of requests through the continuous-batching server;
* ``paths``     ``query_paths``: whole shortest paths.

Graphs (the generators of ``paper_1503_07192_amd.workloads`` at other sizes and
seeds): ``grid`` (4-neighbour grid, uniform weights), ``diag`` (grid plus one
diagonal in half of the cells), ``roads`` (grid with a tenth of the edges
removed and lognormal weights, some vertices cut off), ``delaunay`` (random
points, weights = lengths).  Partitions: square blocks, row by row or along a
Z-order curve, or recursive coordinate bisection; the blocks at the rim of a
grid are smaller when its side is no multiple of the block's.
"""
import numpy as np
import torch

from paper_1503_07192_amd import spq
from paper_1503_07192_amd import workloads as W

OPTIONS = ("bg_method", "group_comps", "level3_groups", "share_comps")


def listed():
    return [
        # one distance for one caller on a small city map: pure call latency
        dict(name="pair_host", op="host", graph="grid", side=32, block=8, wmax=100, q=1),
        # a small batch on the same map, pairs already on the device
        dict(name="batch_small", op="batch", graph="grid", side=32, block=8, wmax=100, q=1000),
        # bulk distances (an origin-destination matrix) on a regional map built
        # with the default options: small blocks, 3 KB read per pair
        dict(name="batch_region", op="batch", graph="diag", side=256, block=8, wmax=1000,
             q=100_000),
        # the same in millions on a map with large components: 14 KB per pair,
        # disconnected vertices among the pairs
        dict(name="batch_bulk", op="batch", graph="roads", side=512, block=16, zorder=True,
             q=2_000_003),
        # an application without device memory of its own: odd batch size, uneven components
        dict(name="batch_host", op="host", graph="delaunay", n=100_003, depth=9, q=50_001),
        # many clients at once: 256 requests of 1 .. 4,096 pairs through the server
        dict(name="serve_burst", op="serve", graph="delaunay", n=100_003, depth=9, requests=256,
             max_log2=12.0),
        # turn-by-turn routes: whole paths of a few hundred vertices
        dict(name="paths_region", op="paths", graph="diag", side=256, block=8, wmax=1_000_000,
             q=500, max_len=2048),
        # the smallest index: launches and host work count, not the kernels
        dict(name="build_city", op="build", graph="grid", side=32, block=8, wmax=100, q=1000),
        # a regional index with the default options
        dict(name="build_region", op="build", graph="diag", side=256, block=8, wmax=1000,
             q=100_000),
        # a large irregular index, ragged components, the autotuner's group size
        # for Delaunay graphs; total weight past int32, so the build certifies itself
        dict(name="build_country", op="build", graph="delaunay", n=400_000, depth=11,
             bg_method=2, group_comps=16, q=100_000),
        # one GPU's share of an index too large for one GPU, the options that
        # the autotuner picks for shares
        dict(name="build_share", op="build", graph="roads", side=1024, block=16, zorder=True,
             share_comps=512, bg_method=2, group_comps=16, level3_groups=8, q=1_000_000),
        # traffic update: all weights of a captured index replaced
        dict(name="reweight_region", op="reweight", graph="diag", side=256, block=8, wmax=1000,
             bg_method=2, group_comps=64, q=100_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    op = rng.choice(["build", "build", "build", "batch", "batch", "host", "serve", "paths",
                     "reweight"])
    c = dict(op=op)
    kind = rng.choice(["grid", "diag", "roads", "delaunay"])
    c["graph"] = kind
    if kind == "delaunay":
        c["n"] = _log_int(rng, 2_000, 150_000)
        # components of about 60 .. 1,000 vertices
        c["depth"] = max(1, int(np.log2(c["n"] / rng.choice([60, 120, 250, 500, 1000]))))
        vbg = 3.9 * c["n"] / np.sqrt(c["n"] / 2 ** c["depth"])
    else:
        c["side"] = _log_int(rng, 20, 260)
        c["block"] = rng.choice([4, 6, 8, 9, 16, 25, 32, 50, 64])
        # the default (flat) closure at most as large as the listed one
        while 4.0 * c["side"] ** 2 / c["block"] > 27_000:
            c["block"] += 1
        c["zorder"] = rng.random() < 0.5
        if kind != "roads":
            c["wmax"] = rng.choice([100, 1000])
        vbg = 4.0 * c["side"] ** 2 / c["block"]
    if rng.random() < 0.4 or op == "reweight" or vbg > 27_000:
        c["bg_method"] = 2
        c["group_comps"] = rng.choice([0, 8, 16, 32])
    if op == "paths":
        # weights fine enough that shortest paths are unique
        c["q"] = _log_int(rng, 1, 400)
        c["max_len"] = 2048
        if "wmax" in c:
            c["wmax"] = 100_000
        if kind == "roads":
            c["wscale"] = 1_000
    elif op == "serve":
        c["requests"] = rng.randint(16, 200)
        c["max_log2"] = rng.choice([4.0, 8.0, 12.0])
    else:
        c["q"] = _log_int(rng, 1, 500_000)
    if op == "build" and kind == "roads" and rng.random() < 0.5:
        k = (-(-c["side"] // c["block"])) ** 2
        if k >= 8:
            c.update(bg_method=2, group_comps=rng.choice([4, 8, 16]), share_comps=max(1, k // 4))
    return c


# ------------------------------------------------------------------ inputs
def _graph(case, seed):
    """(n, eu, ev, w, part, k), numpy int32, drawn from the seed."""
    if case["graph"] == "delaunay":
        g = W.delaunay_graph(case["n"], cfg=1000 + seed, depth=case["depth"])
        return g["n"], g["eu"], g["ev"], g["w"], g["part"], g["k"]
    rng = np.random.default_rng([W.SEED_BASE, seed])
    s = case["side"]
    eu, ev = W.grid_edges(s, s)
    if case["graph"] == "diag":
        r, c = (x.ravel() for x in np.meshgrid(np.arange(s - 1), np.arange(s - 1), indexing="ij"))
        take = rng.random(r.size) < 0.5
        r, c, o = r[take], c[take], rng.integers(0, 2, r.size)[take]
        eu = np.concatenate([eu, (r * s + c + o).astype(np.int32)])
        ev = np.concatenate([ev, ((r + 1) * s + c + 1 - o).astype(np.int32)])
    if case["graph"] == "roads":
        keep = rng.random(len(eu)) >= 0.1
        eu, ev = eu[keep], ev[keep]
        w = np.exp(4.0 + rng.standard_normal(len(eu)))
        w = np.rint(case.get("wscale", 1) * np.clip(w, 1, 1e5)).astype(np.int32)
    else:
        w = rng.integers(1, case["wmax"] + 1, len(eu)).astype(np.int32)
    b = case["block"]
    part, k = W.block_partition(s, s, b, b, 0 if case.get("zorder") else 1)
    return s * s, eu, ev, w, part, k


def _options(case):
    return {o: case[o] for o in OPTIONS if case.get(o)}


def _pairs(case, seed, n, part, q):
    rng = np.random.default_rng([W.SEED_BASE + 1, seed])
    v2 = rng.integers(0, n, q).astype(np.int32)
    if case.get("share_comps"):  # a share answers for its own vertices
        own = np.flatnonzero(part < case["share_comps"]).astype(np.int32)
        return own[rng.integers(0, len(own), q)], v2
    return rng.integers(0, n, q).astype(np.int32), v2


def _requests(case, seed, n, part):
    rng = np.random.default_rng([W.SEED_BASE + 2, case["requests"]])
    sizes = np.floor(2.0 ** rng.uniform(0.0, case["max_log2"], case["requests"])).astype(np.int64)
    v1, v2 = _pairs(case, seed, n, part, int(sizes.sum()))
    cut = np.cumsum(sizes)[:-1]
    return list(zip(np.split(v1, cut), np.split(v2, cut)))


def _device(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def prepare(case, seed):
    n, eu, ev, w, part, k = _graph(case, seed)
    op = case["op"]
    s = dict(op=op, n=n, k=k, opts=_options(case))
    s["eu"], s["ev"], s["w"], s["part"] = (_device(a) for a in (eu, ev, w, part))
    if op != "build":
        extra = {"paths": {"paths": True}, "reweight": {"graph": True}}.get(op, {})
        s["index"] = spq.build_index(n, s["eu"], s["ev"], s["w"], s["part"], k, **s["opts"],
                                     **extra)
    if op == "reweight":  # the new weights: the old ones redrawn edge by edge
        s["w"] = _device(np.random.default_rng([W.SEED_BASE + 3, seed]).permutation(w))
    if op == "serve":
        s["requests"] = _requests(case, seed, n, part)
        s["server"] = spq.Server(s["index"])
    else:
        v1, v2 = _pairs(case, seed, n, part, case["q"])
        if op != "host":
            v1, v2 = _device(v1), _device(v2)
        s["v1"], s["v2"] = v1, v2
        s["max_len"] = case.get("max_len")
    return s


def run(s):
    op = s["op"]
    if op == "build":
        index = spq.build_index(s["n"], s["eu"], s["ev"], s["w"], s["part"], s["k"], **s["opts"])
        out = spq.query_batch(index, s["v1"], s["v2"])
        index.free()
        return out
    if op == "reweight":
        spq.reweight(s["index"], s["w"])
        return spq.query_batch(s["index"], s["v1"], s["v2"])
    if op == "batch":
        return spq.query_batch(s["index"], s["v1"], s["v2"])
    if op == "host":
        return spq.query_batch_host(s["index"], s["v1"], s["v2"])
    if op == "serve":
        tickets = [s["server"].submit(a, b) for a, b in s["requests"]]
        return np.concatenate([s["server"].poll(t, wait=True)[0] for t in tickets])
    return spq.query_paths(s["index"], s["v1"], s["v2"], s["max_len"])


# -------------------------------------------------------------------- work
def work(case):
    """Each input read once and each result written once.  A build's results
    are its tables: every component's distances and the boundary distances
    (one direction per pair, a share's rows in full).  A pair reads a row piece
    per endpoint and the block between the two components."""
    n, eu, ev, w, part, k = _graph(case, 0)
    m = len(eu)
    cross = part[eu] != part[ev]
    boundary = np.zeros(n, bool)
    boundary[eu[cross]] = True
    boundary[ev[cross]] = True
    size = np.bincount(part, minlength=k).astype(np.float64)
    nb = np.bincount(part[boundary], minlength=k).astype(np.float64)
    v = nb.sum()
    mean = float((nb * size).sum() / size.sum())  # |B(C)| of a random vertex
    if case["op"] == "serve":
        q = sum(len(a) for a, _ in _requests(case, 0, n, part))
    else:
        q = case["q"]
    bytes_ = q * (4.0 * (2 * mean + mean * mean) + 28)
    flops = q * 2.0 * mean * mean
    if case["op"] in ("build", "reweight"):
        rows = nb[:case["share_comps"]].sum() if case.get("share_comps") else v / 2
        bytes_ += 12.0 * m + 4.0 * n + 4.0 * (size * size).sum() + 4.0 * rows * v
    if case["op"] == "paths":
        bytes_ += 4.0 * q * case["max_len"]
    return {"bytes": float(bytes_), "flops": float(flops)}


def exact(case, seed):
    """Distances by a plain Floyd-Warshall in int64; small graphs only (paths
    are not unique and have no such value)."""
    n, eu, ev, w, part, k = _graph(case, seed)
    if n > 1024 or case["op"] == "paths":
        return None
    if case["op"] == "reweight":
        w = np.random.default_rng([W.SEED_BASE + 3, seed]).permutation(w)
    inf = np.int64(spq.SPQ_INF)
    d = np.full((n, n), inf)
    np.minimum.at(d, (eu, ev), w.astype(np.int64))
    np.minimum.at(d, (ev, eu), w.astype(np.int64))
    d[np.arange(n), np.arange(n)] = 0
    for x in range(n):
        np.minimum(d, d[:, x:x + 1] + d[x:x + 1, :], out=d)
    np.minimum(d, inf, out=d)
    if case["op"] == "serve":
        return np.concatenate([d[a, b] for a, b in _requests(case, seed, n, part)])
    v1, v2 = _pairs(case, seed, n, part, case["q"])
    return d[v1, v2]
