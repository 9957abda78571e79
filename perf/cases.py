"""What is measured: BFS and SSSP solves through the Python entry points.

A pass is one call as a program that keeps its graph in device memory makes
it: ``lbg.bfs`` / ``lbg.sssp`` from one source, ``lbg.batch_solve`` over many
packed graphs, or a run of ``lbg.Engine`` over a list of requests.  A state is
the graph, the source (or queries), the result tensor and the workspace; all
are made on the GPU from the seed.  The graph families are those of
``graphgen`` (uniform out-degree, R-MAT, road-like grid) with the same
parameters, generated with torch so that new graphs are quick to make.
"""
from __future__ import annotations

import math
import random

import torch

from paper_1711_00231_amd import lbg

DEV = "cuda"
BFS_INF = 2**31 - 1
SSSP_INF = 2**32 - 1


def listed():
    return [
        # The smallest calls: a whole solve of a 16 K-node graph (131 K arcs,
        # 7 BFS levels), where launches and read-backs are most of the time.
        {"name": "bfs_uniform_14", "do": "bfs", "family": "uniform", "n": 1 << 14},
        {"name": "sssp_uniform_14", "do": "sssp", "family": "uniform", "n": 1 << 14, "layout": "csr"},
        # An ordinary directed graph of no round size (8 M arcs).
        {"name": "bfs_uniform_1000003", "do": "bfs", "family": "uniform", "n": 1000003},
        # A ragged skewed graph on the plain CSR arrays, as a program that
        # has just loaded it solves it (9 M arcs).
        {"name": "sssp_rmat_300007", "do": "sssp", "family": "rmat", "n": 300007, "layout": "csr"},
        # The headline graph: R-MAT scale 22, BFS on the CSR arrays and SSSP
        # on the degree-class ordered copy that a resident graph keeps.
        {"name": "bfs_rmat_22", "do": "bfs", "family": "rmat", "n": 1 << 22},
        {"name": "sssp_rmat_22_ordered", "do": "sssp", "family": "rmat", "n": 1 << 22, "layout": "ordered"},
        # The largest resident graph of the serving set (0.5 G arcs).
        {"name": "bfs_rmat_24", "do": "bfs", "family": "rmat", "n": 1 << 24},
        # Road-like: a grid with 1 % long-range shortcuts (55 levels)...
        {"name": "bfs_grid_2048", "do": "bfs", "family": "grid", "width": 2048, "height": 2048, "shortcuts": 0.01},
        {"name": "sssp_grid_2048", "do": "sssp", "family": "grid", "width": 2048, "height": 2048, "shortcuts": 0.01,
         "layout": "csr"},
        # ... and without, thousands of levels of a few thousand nodes each.
        {"name": "sssp_road_2048", "do": "sssp", "family": "grid", "width": 2048, "height": 2048, "shortcuts": 0.0,
         "layout": "csr"},
        # Many graphs at once: 256 instances of uneven size, half R-MAT and
        # half uniform, 4 sources each, BFS and SSSP: 2,048 solves.
        {"name": "batch_256", "do": "batch", "instances": 256, "lo": 10, "hi": 18, "sources": 4},
        # Serving: 48 requests (70 % BFS) over 12 uploaded graphs, admitted
        # into 24 slots as earlier ones finish.
        {"name": "engine_48", "do": "engine", "instances": 12, "lo": 12, "hi": 16, "requests": 48, "slots": 24},
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("uniform", "uniform", "rmat", "rmat", "rmat", "grid", "grid", "batch", "engine"))
    if kind == "batch":
        lo = rng.randint(8, 13)
        return {"do": "batch", "instances": _log_uniform(rng, 8, 192), "lo": lo, "hi": rng.randint(lo + 2, 17),
                "sources": rng.randint(1, 4)}
    if kind == "engine":
        return {"do": "engine", "instances": rng.randint(3, 16), "lo": rng.randint(10, 13), "hi": rng.randint(14, 16),
                "requests": rng.randint(12, 64), "slots": rng.randint(6, 32)}
    do = rng.choice(("bfs", "sssp"))
    case = {"do": do, "family": kind}
    if kind == "grid":
        case["shortcuts"] = rng.choice((0.01, 0.01, 0.0))
        case["width"] = _log_uniform(rng, 100, 2047)
        case["height"] = _log_uniform(rng, 100, 2047)
    else:
        case["n"] = _log_uniform(rng, 1 << 12, 1 << 22)
    if do == "sssp":
        case["layout"] = rng.choice(("csr", "ordered", "packed")) if kind == "rmat" else "csr"
    return case


# ------------------------------------------------------------------ graphs --
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) & 0x7FFFFFFFFFFFFFFF)
    return g


def _mix(x):
    """A 64-bit integer hash (wrapping), as a non-negative value."""
    x = (x ^ (x >> 31)) * 0x4BE98134A5976FD3
    x = (x ^ (x >> 29)) * 0x3BBF2A98B9ADF421
    return (x ^ (x >> 32)) & 0x7FFFFFFFFFFFFFFF


def _symmetric(u, v, n, wmax, salt):
    """CSR of the undirected graph of the pairs (u, v): both directions, no
    self-loops, no duplicates, rows sorted, one weight in [1, wmax] per pair."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.unique(torch.cat((u * n + v, v * n + u)))
    src, dst = key // n, key % n
    w = 1 + _mix(torch.minimum(src, dst) * n + torch.maximum(src, dst) + salt) % wmax
    return _csr(src, n), dst.to(torch.int32), w.to(torch.int32)


def _csr(sorted_src, n):
    off = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(sorted_src, minlength=n), 0, out=off[1:])
    return off.to(torch.int32)


def _uniform(n, wmax, g):
    src = torch.arange(n, device=DEV).repeat_interleave(8)
    dst = torch.randint(0, n, (8 * n,), generator=g, device=DEV)
    keep = src != dst
    src, dst = src[keep], dst[keep]
    w = torch.randint(1, wmax + 1, (dst.numel(),), generator=g, device=DEV, dtype=torch.int32)
    return _csr(src, n), dst.to(torch.int32), w


def _rmat(n, g):
    """R-MAT (.57, .19, .19, .05), 16 n pairs, ids relabelled; for an n that
    is no power of two the pairs with an id beyond n are drawn out."""
    scale = max(1, (n - 1).bit_length())
    full = 1 << scale
    pairs = 16 * full
    u = torch.zeros(pairs, dtype=torch.int64, device=DEV)
    v = torch.zeros(pairs, dtype=torch.int64, device=DEV)
    for _ in range(scale):
        r = torch.rand(pairs, generator=g, device=DEV)
        u = 2 * u + (r >= 0.76)
        v = 2 * v + (((r >= 0.57) & (r < 0.76)) | (r >= 0.95))
    perm = torch.randperm(full, generator=g, device=DEV)
    u, v = perm[u], perm[v]
    if full != n:
        keep = (u < n) & (v < n)
        u, v = u[keep], v[keep]
    salt = int(torch.randint(0, 1 << 40, (1,), generator=g, device=DEV))
    return _symmetric(u, v, n, 255, salt)


def _grid(width, height, shortcuts, g):
    n = width * height
    node = torch.arange(n, device=DEV)
    right = node[node % width < width - 1]
    down = node[: n - width]
    u = torch.cat((right, down))
    v = torch.cat((right + 1, down + width))
    keep = torch.rand(u.numel(), generator=g, device=DEV) >= 0.1
    u, v = u[keep], v[keep]
    extra = int(shortcuts * u.numel())
    if extra:
        ends = torch.randint(0, n, (2, extra), generator=g, device=DEV)
        u, v = torch.cat((u, ends[0])), torch.cat((v, ends[1]))
    salt = int(torch.randint(0, 1 << 40, (1,), generator=g, device=DEV))
    return _symmetric(u, v, n, 1000, salt)


def _rmat_arcs(n):
    """About how many arcs _rmat has after its duplicates are gone."""
    scale = max(1, (n - 1).bit_length())
    return int(32 * (1 - 1.1 * 2 ** (-scale / 5.2)) * (n * n >> scale))


def _instances(case):
    """(family, n) of the instances of a batch or an engine: by the case."""
    rng = random.Random(1000 * case["lo"] + case["hi"])
    if case["do"] == "engine":
        return [("uniform", int(2 ** rng.uniform(case["lo"], case["hi"]))) for _ in range(case["instances"])]
    return [("rmat", 1 << rng.randint(case["lo"], case["hi"])) if i % 2 == 0
            else ("uniform", int(2 ** rng.uniform(case["lo"], case["hi"]))) for i in range(case["instances"])]


def _packed(sizes, g):
    """One CSR of the instances' disjoint union, and the first node of each."""
    offs, cols, ws, base, arcs = [], [], [], [0], 0
    for family, n in sizes:
        o, c, w = _rmat(n, g) if family == "rmat" else _uniform(n, 255, g)
        offs.append(o[:-1] + arcs)
        cols.append(c + base[-1])
        ws.append(w)
        base.append(base[-1] + n)
        arcs += c.numel()
    offs.append(torch.tensor([arcs], dtype=torch.int32, device=DEV))
    return torch.cat(offs), torch.cat(cols), torch.cat(ws), base


def _sources(offsets, lo, hi, count, g):
    """Random nodes of [lo, hi) that have out-arcs."""
    deg = offsets[lo + 1: hi + 1] - offsets[lo:hi]
    at = torch.nonzero(deg > 0).flatten()
    pick = torch.randint(0, at.numel(), (count,), generator=g, device=DEV)
    return [lo + int(x) for x in at[pick].cpu()]


def _queries(case, offsets, base, g):
    """(source, first node, end node, kind) of every solve of the case."""
    k = len(base) - 1
    if case["do"] == "batch":  # sources x kinds, each over every instance
        src = [_sources(offsets, base[i], base[i + 1], case["sources"], g) for i in range(k)]
        return [(src[i][j], base[i], base[i + 1], kind) for kind in (lbg.KIND_BFS, lbg.KIND_SSSP)
                for j in range(case["sources"]) for i in range(k)]
    rng = random.Random(case["requests"])  # which instance and kind each request has
    asked = [(rng.randrange(k), lbg.KIND_BFS if rng.random() < 0.7 else lbg.KIND_SSSP)
             for _ in range(case["requests"])]
    return [(_sources(offsets, base[i], base[i + 1], 1, g)[0], base[i], base[i + 1], kind) for i, kind in asked]


def _inputs(case, seed):
    """(offsets, cols, weights, source or queries) of the case."""
    g = _gen(seed)
    if case["do"] in ("batch", "engine"):
        off, cols, w, base = _packed(_instances(case), g)
        return off, cols, w, _queries(case, off, base, g)
    if case["family"] == "uniform":
        off, cols, w = _uniform(case["n"], 100, g)
    elif case["family"] == "rmat":
        off, cols, w = _rmat(case["n"], g)
    else:
        off, cols, w = _grid(case["width"], case["height"], case["shortcuts"], g)
    return off, cols, w, _sources(off, 0, off.numel() - 1, 1, g)[0]


# ------------------------------------------------------------------- cases --
def prepare(case, seed):
    off, cols, w, asked = _inputs(case, seed)
    do = case["do"]
    graph = lbg.DeviceGraph(off, cols, None if do == "bfs" else w)
    st = {"do": do, "graph": graph, "asked": asked}
    if do == "engine":
        rows, at = [], 0
        for _, lo, hi, _ in asked:
            rows.append(at)
            at += hi - lo
        st["rows"], st["slots"] = rows, case["slots"]
        # room for every slot on the largest instance
        biggest = max(int(off[hi]) - int(off[lo]) for _, lo, hi, _ in asked)
        st["engine"] = lbg.Engine(graph, case["slots"], at, case["slots"] * biggest)
        return st
    st["workspace"] = lbg.Workspace(DEV)
    if do == "batch":
        graph.host_offsets = off.cpu().numpy()
        st["out"] = torch.empty(sum(hi - lo for _, lo, hi, _ in asked), dtype=torch.int32, device=DEV)
    else:
        st["out"] = torch.empty(graph.n, dtype=torch.int32, device=DEV)
        st["layout"] = case.get("layout", "csr")
        if st["layout"] == "ordered":
            graph.ensure_ordered()
        elif st["layout"] == "packed":
            graph.ensure_packed()
    return st


def _serve(st):
    """Requests into slots as they come free, two levels at a time."""
    eng, asked, rows = st["engine"], st["asked"], st["rows"]
    nxt, running = 0, 0
    while nxt < len(asked) or running:
        while nxt < len(asked) and running < st["slots"]:
            eng.submit(*asked[nxt], rows[nxt])
            nxt += 1
            running += 1
        for slot in eng.step(2):
            eng.release(slot)
            running -= 1
    return eng.rows


def run(state):
    do = state["do"]
    if do == "bfs":
        return lbg.bfs(state["graph"], state["asked"], out=state["out"], workspace=state["workspace"])
    if do == "sssp":
        return lbg.sssp(state["graph"], state["asked"], out=state["out"], workspace=state["workspace"],
                        ordered=state["layout"] == "ordered", packed=state["layout"] == "packed")
    if do == "batch":
        return lbg.batch_solve(state["graph"], state["asked"], out=state["out"], workspace=state["workspace"])
    return _serve(state)


def work(case):
    """Bytes: the offsets, columns and (SSSP) weights once per graph, and the
    results once.  Operations: one comparison per arc and solve."""
    do = case["do"]
    if do in ("batch", "engine"):
        sizes = _instances(case)
        n = [s for _, s in sizes]
        m = [_rmat_arcs(s) if f == "rmat" else 8 * s for f, s in sizes]
        if do == "batch":
            solves = [2 * case["sources"]] * len(n)
        else:
            rng = random.Random(case["requests"])
            solves = [0] * len(n)
            for _ in range(case["requests"]):
                solves[rng.randrange(len(n))] += 1
                rng.random()
        graph = sum(4 * a + 8 * b for a, b, s in zip(n, m, solves) if s)
        return {"bytes": graph + sum(4 * a * s for a, s in zip(n, solves)),
                "flops": sum(b * s for b, s in zip(m, solves))}
    if case["family"] == "grid":
        n = case["width"] * case["height"]
        m = int(3.6 * n * (1 + case["shortcuts"]))
    else:
        n = case["n"]
        m = 8 * n if case["family"] == "uniform" else _rmat_arcs(n)
    return {"bytes": 8 * n + (4 if do == "bfs" else 8) * m, "flops": m}


# ------------------------------------------------------------------- exact --
def _relaxed(src, dst, w, source, n):
    """Distances over 64-bit sums: relax every arc until nothing changes."""
    far = 1 << 60
    d = torch.full((n,), far, dtype=torch.int64, device=DEV)
    d[source] = 0
    while True:
        nd = d.scatter_reduce(0, dst, d[src] + w, "amin")
        if torch.equal(nd, d):
            return torch.where(d < far, d, -1)
        d = nd


def exact(case, seed):
    """The same rows from plain torch in 64 bits; None for the grids without
    shortcuts (thousands of relaxations of every arc)."""
    if case.get("shortcuts") == 0.0:
        return None
    off, cols, w, asked = _inputs(case, seed)
    off, n = off.to(torch.int64), off.numel() - 1
    src = torch.arange(n, device=DEV).repeat_interleave(off[1:] - off[:-1])
    dst, w = cols.to(torch.int64), w.to(torch.int64)

    def rows(d, bfs):  # unreachable: INT32_MAX levels, UINT32_MAX bits
        return torch.where(d < 0, BFS_INF, d).to(torch.int32) if bfs else d.to(torch.int32)

    if case["do"] in ("bfs", "sssp"):
        bfs = case["do"] == "bfs"
        return rows(_relaxed(src, dst, torch.ones_like(w) if bfs else w, asked, n), bfs)
    if case["do"] == "batch":  # the queries come in runs of one solve per instance
        k = case["instances"]
        out = []
        for j in range(0, len(asked), k):
            q = asked[j: j + k]
            bfs = q[0][3] == lbg.KIND_BFS
            at = torch.tensor([s for s, _, _, _ in q], device=DEV)
            out.append(rows(_relaxed(src, dst, torch.ones_like(w) if bfs else w, at, n), bfs))
        return torch.cat(out)
    out = []
    for s, lo, hi, kind in asked:
        a, b = int(off[lo]), int(off[hi])
        bfs = kind == lbg.KIND_BFS
        ww = torch.ones_like(w[a:b]) if bfs else w[a:b]
        out.append(rows(_relaxed(src[a:b] - lo, dst[a:b] - lo, ww, s - lo, hi - lo), bfs))
    return torch.cat(out)
