"""The small-frontier team (levels of at most 524,288 arcs run on the device by
up to 128 workgroups) against the oracle, bit for bit, at the sizes where its
cuts fall: one arc per level, hubs that span every workgroup, levels of exactly
the largest size and one arc more, and hand-overs to one-level launches and
back."""
import numpy as np
import pytest

import graphgen
import oracle
import pins

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
from paper_1711_00231_amd import lbg  # noqa: E402

O = oracle.get()
LIMIT = 128 * 4096  # arcs of a level that the team takes


@pytest.fixture(autouse=True)
def _reset():
    yield
    lbg.set_bfs_scan_min(-1)
    lbg.set_addressing(0)


def _fan(width, tail=3, salt=0):
    """A path of 3 nodes into a hub with `width` children; every 7th child
    starts a chain of `tail` nodes, every 11th points back at the hub."""
    rng = np.random.default_rng(salt)
    kids = 4 + np.arange(width)
    src, dst = [np.arange(3), np.full(width, 3)], [np.arange(1, 4), kids]
    nxt = 4 + width
    heads = kids[::7]
    for _ in range(tail):
        new = nxt + np.arange(heads.size)
        src.append(heads)
        dst.append(new)
        heads, nxt = new, nxt + heads.size
    src.append(kids[::11])
    dst.append(np.full(kids[::11].size, 3))
    s, d = np.concatenate(src), np.concatenate(dst)
    perm = rng.permutation(nxt)  # ids in no order
    g = graphgen.from_edges(nxt, perm[s], perm[d], rng.integers(1, 90, s.size), f"fan{width}")
    return g, int(perm[0])


def _cases():
    yield "path", pins.path_graph(300, np.arange(1, 300) % 9), 0
    for width in (1, 63, 64, 2047, 2048, 2049, 4096, 128 * 64, LIMIT - 1, LIMIT, LIMIT + 1):
        yield (f"fan{width}", *_fan(width, salt=width))
    for n, k in ((7, 1), (129, 3), (5000, 8), (40000, 5), (90001, 11)):
        yield f"uniform{n}x{k}", graphgen.uniform(n=n, k=k, salt=n), 1
    yield "grid150", graphgen.grid(150, 97, shortcut_frac=0), 60
    yield "rmat14", graphgen.rmat(14), int(graphgen.sources(graphgen.rmat(14), 1, graphgen.FAMILY_RMAT)[0])


CASES = list(_cases())


@pytest.mark.parametrize("limit", [-1, 2, 700, 33000])
@pytest.mark.parametrize("wide", [0, 1])
def test_team_levels(limit, wide):
    """limit: levels of at least so many arcs leave the team (-1: the
    default, LIMIT + 1); 33000 lies just above the size up to which every
    arc issues its atomic without reading first."""
    lbg.set_bfs_scan_min(limit)
    lbg.set_addressing(wide)
    ws = lbg.Workspace()
    for name, g, s in CASES:
        dg = lbg.DeviceGraph.from_numpy(g.offsets, g.cols, g.weights)
        exp_l = O.bfs(g.offsets, g.cols, s)
        exp_d = O.dijkstra(g.offsets, g.cols, g.weights, s)
        got, st = lbg.bfs(dg, s, workspace=ws, stats=True)
        assert np.array_equal(got.cpu().numpy(), exp_l), (name, "bfs")
        reached = exp_l != pins.BFS_INF
        assert st["updates"] == int(reached.sum()) - 1, (name, st)
        assert st["edges_scanned"] == g.reached_arcs(reached), (name, st)
        for kw in ({}, {"packed": True}, {"ordered": True}):
            d = lbg.sssp(dg, s, workspace=ws, **kw).cpu().numpy().view(np.uint32)
            assert np.array_equal(d, exp_d), (name, "sssp", kw)


def test_team_limit_boundary():
    """A level of exactly LIMIT arcs runs in the team, one arc more does not."""
    for width, one_level in ((LIMIT, 0), (LIMIT + 1, 1)):
        g, s = _fan(width, tail=0)
        dg = lbg.DeviceGraph.from_numpy(g.offsets, g.cols, g.weights)
        lbg.profile_enable(True, reset=True)
        lv = lbg.bfs(dg, s)
        lbg.profile_enable(False, reset=False)
        assert np.array_equal(lv.cpu().numpy(), O.bfs(g.offsets, g.cols, s))
        assert lbg.profile_read("bfs_small")["launches"] >= 1
        assert (lbg.profile_read("bfs")["launches"] > 0) == bool(one_level), width


def test_teams_side_by_side():
    """Solves from several threads and streams at once: teams come together
    with whatever workgroups are scheduled, and every result is exact."""
    import threading

    g = graphgen.grid(400, 300, shortcut_frac=0)
    h = graphgen.uniform(15)
    jobs = [(g, 5), (h, 9), (g, 70000), (h, 1)]
    exp = [(O.bfs(x.offsets, x.cols, s), O.dijkstra(x.offsets, x.cols, x.weights, s)) for x, s in jobs]
    dgs = {id(x): lbg.DeviceGraph.from_numpy(x.offsets, x.cols, x.weights) for x in (g, h)}
    bad = []

    def work(k):
        try:
            x, s = jobs[k]
            st = torch.cuda.Stream()
            ws = lbg.Workspace()
            for _ in range(4):
                lv = lbg.bfs(dgs[id(x)], s, workspace=ws, stream=st)
                d = lbg.sssp(dgs[id(x)], s, workspace=ws, stream=st)
                st.synchronize()
                if not np.array_equal(lv.cpu().numpy(), exp[k][0]):
                    bad.append((k, "bfs"))
                if not np.array_equal(d.cpu().numpy().view(np.uint32), exp[k][1]):
                    bad.append((k, "sssp"))
        except Exception as e:  # reported below
            bad.append(repr(e))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(100)
    assert not any(t.is_alive() for t in ts)
    assert not bad, bad


@pytest.mark.parametrize("layout", ["csr", "packed", "ordered"])
def test_near_far(layout):
    """SSSP solves that defer far nodes (at least 2^20 arcs, at most 16 per
    node): long paths, gaps far beyond the threshold step, all weights zero,
    equal weights, and one weight that dwarfs the others."""
    rng = np.random.default_rng(7)
    road = graphgen.grid(640, 520, shortcut_frac=0)
    uni = graphgen.uniform(n=140_000, k=8, salt=3)
    graphs = [(road, 77), (graphgen.grid(600), 4), (uni, 11)]
    for w in (np.zeros(uni.m), np.full(uni.m, 7), np.where(rng.random(uni.m) < 1e-4, 90_000, 1),
              np.where(np.arange(uni.m) % 8 == 0, 1, 200)):
        graphs.append((graphgen.Graph("w", uni.offsets, uni.cols, w.astype(np.uint32)), 11))
    # two halves joined by one heavy arc: the far set is empty of near nodes
    # until the threshold has jumped the gap
    half = graphgen.uniform(n=70_000, k=8, salt=9)
    off = np.concatenate([half.offsets, half.offsets[1:] + half.m]).astype(np.int32)
    cols = np.concatenate([half.cols, half.cols + half.n]).astype(np.int32)
    w = np.concatenate([half.weights, half.weights]).astype(np.uint32)
    k = int(half.offsets[1234])
    cols[k], w[k] = half.n + 5, 4_000_000
    graphs.append((graphgen.Graph("gap", off, cols, w), 3))
    ws = lbg.Workspace()
    for g, s in graphs:
        assert (1 << 20) <= g.m <= 16 * g.n
        dg = lbg.DeviceGraph.from_numpy(g.offsets, g.cols, g.weights)
        if layout == "packed" and int(g.weights.max()) > 8191:
            continue  # ids and weights do not fit one word
        exp = O.dijkstra(g.offsets, g.cols, g.weights, s)
        for wide in (0, 1):
            lbg.set_addressing(wide)
            d, st = lbg.sssp(dg, s, workspace=ws, packed=layout == "packed", ordered=layout == "ordered", stats=True)
            assert np.array_equal(d.cpu().numpy().view(np.uint32), exp), (g.name, s, wide)
            assert st["edges_scanned"] >= g.reached_arcs(exp != 0xFFFFFFFF)


@pytest.mark.parametrize("path_len", [1, 2, 40])
def test_many_team_launches(path_len):
    """A chain of ten dense blocks joined by paths: big levels run as one-level
    launches, the paths in the team, so a solve makes many team launches, some
    of which find nothing to do; each has to find its control words cleared by
    the launches before it, whether those ran a level or not."""
    parts_s, parts_d, base, n_mid = [], [], 0, 60_000
    for b in range(10):
        ids = base + np.arange(path_len)
        if b:
            parts_s.append([base - 1]); parts_d.append([base])
        parts_s.append(ids[:-1]); parts_d.append(ids[1:])
        base += path_len
        blk = graphgen.uniform(n=n_mid, k=24, salt=70 + b)
        parts_s.append([base - 1]); parts_d.append([base])
        parts_s.append(base + np.repeat(np.arange(n_mid), blk.degrees)); parts_d.append(base + blk.cols.astype(np.int64))
        base += n_mid
    s, d = np.concatenate(parts_s), np.concatenate(parts_d)
    w = np.random.default_rng(path_len).integers(1, 60, s.size)
    for wts in (w, np.ones_like(w)):
        g = graphgen.from_edges(base, s, d, wts, "chain")
        dg = lbg.DeviceGraph.from_numpy(g.offsets, g.cols, g.weights)
        assert np.array_equal(lbg.bfs(dg, 0).cpu().numpy(), O.bfs(g.offsets, g.cols, 0))
        exp = O.dijkstra(g.offsets, g.cols, g.weights, 0)
        for kw in ({}, {"ordered": True}):
            assert np.array_equal(lbg.sssp(dg, 0, **kw).cpu().numpy().view(np.uint32), exp), kw


@pytest.mark.parametrize("solve", ["bfs", "sssp"])
def test_teams_beside_big_levels(solve):
    """Team launches of several streams while big levels of others hold the
    CUs, XCD by XCD: a team's first workgroup may start after the team has
    come together without it, run its levels and ended, and must then leave
    the next level alone."""
    import threading

    big = graphgen.rmat(18)
    small = graphgen.grid(256, shortcut_frac=0)
    mid = graphgen.uniform(16)
    srcs = graphgen.sources(big, 2, graphgen.FAMILY_RMAT)
    jobs = [(big, int(srcs[0])), (small, 9), (big, int(srcs[1])), (mid, 4), (mid, 77), (small, 3000)]
    if solve == "bfs":
        exp = [O.bfs(x.offsets, x.cols, s) for x, s in jobs]
    else:
        exp = [O.dijkstra(x.offsets, x.cols, x.weights, s) for x, s in jobs]
    dgs = {id(x): lbg.DeviceGraph.from_numpy(x.offsets, x.cols, x.weights) for x in (big, small, mid)}
    bad = []

    def work(k):
        try:
            x, s = jobs[k]
            st = torch.cuda.Stream()
            ws = lbg.Workspace()
            for i in range(24):
                out = getattr(lbg, solve)(dgs[id(x)], s, workspace=ws, stream=st)
                st.synchronize()
                if not np.array_equal(out.cpu().numpy().view(exp[k].dtype), exp[k]):
                    bad.append((k, i))
        except Exception as e:  # reported below
            bad.append(repr(e))

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(jobs))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(100)
    assert not any(t.is_alive() for t in ts)
    assert not bad, bad


def test_hub_improved_many_times_in_one_level():
    """3,000 parallel arcs of falling weight to a node of 2^26 arcs, which
    every improvement queues again: 64 times its arcs are 2^32."""
    n, k, hub = 1000, 3000, 1 << 26
    off = np.zeros(n + 1, dtype=np.int32)
    off[2:] = k
    off[n] = k + hub
    cols = np.concatenate([np.full(k, n - 1), np.arange(hub, dtype=np.int32) % (n - 1)]).astype(np.int32)
    w = np.concatenate([2 * k - np.arange(k), np.full(hub, 7)]).astype(np.uint32)
    dg = lbg.DeviceGraph.from_numpy(off, cols, w)
    exp = O.dijkstra(off, cols, w, 1)
    ws = lbg.Workspace()
    for _ in range(20):
        got = lbg.sssp(dg, 1, workspace=ws).cpu().numpy().view(np.uint32)
        assert np.array_equal(got, exp)
