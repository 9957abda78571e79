"""The balanced strategy's kernels on the host (tests/c/emul): the team of
workgroups that runs small levels, near-far SSSP and the one-level launches,
compiled from the sources that the library is built from, with a workgroup's
first or second wavefront running ahead of the others and every array ending
at an unmapped page.  Full solves equal the oracle; the cases after them are
inputs on which an earlier form of these kernels was wrong."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import graphgen
import oracle

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
O = oracle.get()
BAD_SRC = 32  # the guard of a source outside the graph


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("team")
    exe = str(d / "team_run")
    # 32-bit sources of 64-lane masks: the warnings the device compiler has not
    subprocess.run(["g++", "-O1", "-std=c++20", "-pthread", "-w", "-I", os.path.join(ROOT, "tests", "c", "emul"),
                    "-I", os.path.join(ROOT, "paper_1711_00231_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c", "emul", "team_run.cpp"), "-o", exe], check=True)

    def run(g, **opt):
        gf, of = str(d / "graph"), str(d / "out")
        w = g.weights if g.weights is not None else np.ones(g.m)
        with open(gf, "wb") as f:
            np.array([g.n, g.m], dtype=np.int32).tofile(f)
            np.asarray(g.offsets, dtype=np.int32).tofile(f)
            np.asarray(g.cols, dtype=np.int32).tofile(f)
            np.asarray(w, dtype=np.uint32).tofile(f)
        r = subprocess.run([exe, gf, of] + [f"{k}={int(v)}" for k, v in opt.items()], capture_output=True, text=True,
                           timeout=300)
        assert r.returncode == 0, (r.returncode, r.stderr[-500:])
        raw = open(of, "rb").read()
        head = np.frombuffer(raw, np.int64, 8)
        st = dict(zip(("error", "levels", "next", "arcs", "entries", "teams", "ones", "plain"), (int(x) for x in head)))
        rest = np.frombuffer(raw, np.uint32, offset=64)
        st["worklist"] = rest[g.n:].reshape(2, -1)  # edge prefixes, first arcs
        return rest[: g.n], st

    return run


def _graphs():
    yield graphgen.uniform(9)
    yield graphgen.grid(24, shortcut_frac=0.02)
    yield graphgen.rmat(9)


@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("far,alone", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_sssp_equals_the_oracle(emu, far, alone, first):
    """alone: the launches that follow a submission without progress, which
    split the far set in the one-level kernel."""
    for g in _graphs():
        s = int(np.argmax(g.degrees))
        for limit in (1 << 20, 300):  # levels in the team; some beyond it
            got, st = emu(g, src=s, far=far, alone=alone, first=first, fill=0x5A, limit=limit, blocks=4)
            assert st["error"] == 0
            assert np.array_equal(got, O.dijkstra(g.offsets, g.cols, g.weights, s)), (g.name, limit)
            assert (st["ones"] > 0) == bool(alone or (limit == 300 and not g.name.startswith("grid"))), g.name
            if alone:
                break


@pytest.mark.parametrize("first", [0, 1])
def test_bfs_equals_the_oracle(emu, first):
    for g in _graphs():
        s = int(np.argmax(g.degrees))
        for limit, alone in ((1 << 20, 0), (300, 0), (300, 1)):
            got, st = emu(g, sssp=0, src=s, alone=alone, first=first, fill=0x5A, limit=limit, blocks=4)
            assert st["error"] == 0
            assert np.array_equal(got.view(np.int32), O.bfs(g.offsets, g.cols, s)), (g.name, limit, alone)


def _graph(n, arcs):
    """A graph of the arcs (u, v, w), in the order given."""
    u, v, w = (np.array(x) for x in zip(*arcs))
    o = np.argsort(u, kind="stable")
    off = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=n))]).astype(np.int32)
    return graphgen.Graph("made", off, v[o].astype(np.int32), w[o].astype(np.uint32))


@pytest.mark.parametrize("hub", [1 << 26, (1 << 26) - 1, 1 << 22, 3])
def test_a_hub_improved_many_times_in_one_level(emu, hub):
    """1,024 parallel arcs of falling weight to a node of `hub` arcs: every
    improvement queues the node, and 64 x 2^26 arcs are 2^32.  The next level
    holds the hub's arcs once."""
    n = 1000
    g = _graph(n, [(1, n - 1, 5000 - k) for k in range(1024)])
    _, st = emu(g, src=1, extra=hub, limit=4096, blocks=8, stop=hub > 4096)
    assert st["error"] == 0
    if hub > 4096:
        assert (st["arcs"], st["entries"]) == (hub, 1)
        assert st["worklist"].tolist() == [[0], [1024]]
    else:
        assert st["arcs"] == 0 and st["next"] > 1


@pytest.mark.parametrize("first", [0, 1])
def test_a_split_whose_nodes_are_all_one_workgroups(emu, first):
    """Nodes that leave the far set together and lie in one workgroup's share
    of it: their arcs are dealt out again right after the split."""
    arcs = [(1000, v, 500_000 + v) for v in range(30)]
    arcs += [(v, 200 + (17 * v + 13 * k) % 800, 1 + k) for v in range(30) for k in range(60)]
    g = _graph(1024, arcs)
    got, st = emu(g, src=1000, far=1, limit=8 * 4096, blocks=8, first=first)
    assert st["error"] == 0
    assert np.array_equal(got, O.dijkstra(g.offsets, g.cols, g.weights, 1000))


@pytest.mark.parametrize("fill,join", [(0xFF, 0), (0x25, 0), (0x00, 1), (0xA5, 0x7FFFFFFF), (0x01, 0x80000003)])
@pytest.mark.parametrize("far", [0, 1])
def test_a_source_renamed_out_of_the_graph(emu, far, fill, join):
    """The call ends with the error at once, whatever the workspace and the
    output (which holds the far set) were left with."""
    g = graphgen.uniform(n=1001, k=8)
    for renamed in (g.n, g.n + 17, -1):
        _, st = emu(g, src=5, renamed=renamed, far=far, fill=fill, join=join, blocks=4)
        assert st["error"] == BAD_SRC


def test_nothing_runs_after_an_error(emu):
    """A team launch behind one that failed leaves everything as it is."""
    g = graphgen.grid(24, shortcut_frac=0.02)
    for far in (0, 1):
        out, st = emu(g, src=5, far=far, blocks=4, error=128, fill=0x5A)
        assert (st["error"], st["levels"], st["next"]) == (128, 0, 0)
        assert st["arcs"] == g.degrees[5]


@pytest.mark.parametrize("weights,plain", [((1, 100), 0), ((1, 10), 0), ((1, 4), 1), ((50, 100), 1), ((7, 7), 1), ((0, 0), 1)])
def test_what_defers_nodes(emu, weights, plain):
    """Weights that hardly differ, and graphs most of whose nodes have next to
    no arcs, defer nothing."""
    g = graphgen.uniform(n=1500, k=8, wlo=weights[0], whi=weights[1], salt=3)
    got, st = emu(g, src=5, far=1, blocks=4, limit=4000)
    assert (st["error"], st["plain"]) == (0, plain)
    assert np.array_equal(got, O.dijkstra(g.offsets, g.cols, g.weights, 5))
    if weights == (1, 100):
        arcs = [(v, (3 * v + k) % 1500, 1 + (7 * k) % 100) for v in range(1500) for k in range(900 if v % 100 == 0 else 1)]
        g = _graph(1500, arcs)
        got, st = emu(g, src=5, far=1, blocks=4, limit=4000)
        assert (st["error"], st["plain"]) == (0, 1)
        assert np.array_equal(got, O.dijkstra(g.offsets, g.cols, g.weights, 5))


@pytest.mark.parametrize("sssp", [0, 1])
def test_tile_marks_of_long_and_short_lists(emu, sssp):
    """A level that leaves the team: entries of one arc up to many tiles."""
    degrees = [1, 2, 511, 512, 513, 1024, 4095, 4096, 4097, 8 * 512, 8 * 512 + 1, 9 * 1024, 70 * 1024 + 5, 3, 1]
    n = 2000
    arcs = [(1, 10 + i, 1) for i in range(len(degrees))]
    arcs += [(10 + i, 100 + k % 1800, 1) for i, d in enumerate(degrees) for k in range(d)]
    g = _graph(n, arcs)
    _, st = emu(g, sssp=sssp, src=1, limit=1000, blocks=3, stop=1)
    assert (st["error"], st["arcs"], st["entries"]) == (0, sum(degrees), len(degrees))


@pytest.mark.parametrize("first", [0, 1])
@pytest.mark.parametrize("tail", [1, 3, 700, 1500])
def test_bfs_levels_of_one_workgroup(emu, first, tail):
    """A path into a fan of `tail` nodes, which meet again in a second path:
    while one workgroup holds the frontier it runs ahead of the others."""
    n = 2 * 1300 + tail
    arcs = [(v, v + 1, 1) for v in range(1299)] + [(v + 1, v, 1) for v in range(1299)]
    arcs += [(1299, 1300 + k, 1) for k in range(tail)] + [(1300 + k, 1300 + tail, 1) for k in range(tail)]
    arcs += [(v, v + 1, 1) for v in range(1300 + tail, n - 1)]
    g = _graph(n, arcs)
    for limit in (1 << 20, 900):
        got, st = emu(g, sssp=0, src=3, first=first, limit=limit, blocks=6)
        exp = O.bfs(g.offsets, g.cols, 3)
        assert st["error"] == 0 and np.array_equal(got.view(np.int32), exp)
        assert st["levels"] == int(exp[g.degrees > 0].max()) + 1
