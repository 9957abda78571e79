"""Batched queries solved by one workgroup each (batches whose arc bound is at
least 2^28) against the oracle, bit for bit: instance sizes around the classes'
LDS sizes, nodes with many arcs (one, and more than the workgroup lists),
instances beyond the arc limit in the same batch, and arcs that leave their
instance."""
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
BOUND = 1 << 28  # arcs of a batch from which small queries run alone; its 256th is their limit


@pytest.fixture(autouse=True)
def _reset():
    yield
    lbg.set_addressing(0)


def _star(n, hubs, salt):
    """`hubs` nodes with arcs to everyone, the others with one arc back."""
    rng = np.random.default_rng(salt)
    src = np.concatenate([np.repeat(np.arange(hubs), n), np.arange(n)])
    dst = np.concatenate([np.tile(np.arange(n), hubs), rng.integers(0, n, n)])
    return graphgen.from_edges(n, src, dst, rng.integers(0, 300, src.size), f"star{hubs}")


def _instances():
    gs = [graphgen.uniform(n=n, k=3, wlo=0, whi=255, salt=n % 251)
          for n in (1, 2, 31, 32, 33, 63, 64, 65, 1000, 8191, 8192, 8193, 32767, 32768, 32769, 262143, 262144, 262145)]
    gs += [_star(2047, 1, 1), _star(2048, 3, 2), _star(4500, 70, 3)]
    gs += [graphgen.rmat(14, salt=3), graphgen.grid(90, 70, shortcut_frac=0), pins.path_graph(500, np.arange(1, 500) % 7)]
    gs += [graphgen.uniform(n=150_000, k=8, salt=8)]  # 1.2 M arcs: beyond the limit
    gs += [graphgen.from_edges(5, [], [], [], "no-arcs")]
    return gs


@pytest.mark.parametrize("wide", [0, 1])
def test_solo_matches_oracle(wide):
    lbg.set_addressing(wide)
    gs = _instances()
    u, nb, _ = graphgen.pack(gs)
    dg = lbg.DeviceGraph.from_numpy(u.offsets, u.cols, u.weights)
    rng = np.random.default_rng(4)
    queries, expect = [], []
    for i, g in enumerate(gs):
        for s in {0, int(rng.integers(g.n)), g.n - 1}:
            for kind in (lbg.KIND_BFS, lbg.KIND_SSSP):
                queries.append((int(nb[i] + s), int(nb[i]), int(nb[i + 1]), kind))
                expect.append((g.name, s, O.bfs(g.offsets, g.cols, s) if kind == lbg.KIND_BFS
                               else O.dijkstra(g.offsets, g.cols, g.weights, s).view(np.int32)))
    ws = lbg.Workspace()
    rows = sum(q[2] - q[1] for q in queries)
    out = torch.full((rows + 7,), -3, dtype=torch.int32, device="cuda")
    for bound in (BOUND, BOUND - 1):  # alone, and all in the shared worklist
        for _ in range(2):
            out.fill_(-3)
            got, st = lbg.batch_solve(dg, queries, out=out, total_arcs=bound, workspace=ws, stats=True)
            got = got.cpu().numpy()
            off = 0
            for q, (name, s, e) in zip(queries, expect):
                assert np.array_equal(got[off: off + e.size], e), (bound, name, s, q[3])
                off += e.size
            assert np.all(got[off:] == -3)
            assert st["levels"] >= 499 and st["edges_scanned"] >= u.m and st["updates"] > 0


def test_solo_rejects_arc_leaving_instance():
    g = graphgen.from_edges(6, [0, 1, 2, 3], [1, 2, 4, 5], [1, 1, 1, 1], "crossing")
    dg = lbg.DeviceGraph.from_numpy(g.offsets, g.cols, g.weights)
    for kind in (lbg.KIND_BFS, lbg.KIND_SSSP):
        with pytest.raises(lbg.LbgError) as ei:
            lbg.batch_solve(dg, [(0, 0, 3, kind), (3, 3, 6, kind)], total_arcs=BOUND)
        assert ei.value.code == lbg.EOVERFLOW


@pytest.mark.parametrize("wide", [0, 1])
def test_solo_batches_of_as_many_arcs(wide):
    """The same instances in batches whose queries hold 2^29 arcs and more, by
    repetition, and one beyond the limit, a 256th of that.  One workgroup's
    atomics are in LDS and not counted: a BFS batch without the large instance
    counts none."""
    lbg.set_addressing(wide)
    gs = _instances() + [graphgen.uniform(n=300_000, k=8, salt=9)]
    u, nb, _ = graphgen.pack(gs)
    dg = lbg.DeviceGraph.from_numpy(u.offsets, u.cols, u.weights)
    for kinds, largest in (((lbg.KIND_BFS, lbg.KIND_SSSP), 1 << 30), ((lbg.KIND_BFS,), 1 << 21)):
        once, expect, arcs = [], [], 0
        for i, g in enumerate(gs):
            for kind in kinds if g.m <= largest else ():
                once.append((int(nb[i] + g.n - 1), int(nb[i]), int(nb[i + 1]), kind))
                expect.append(O.bfs(g.offsets, g.cols, g.n - 1) if kind == lbg.KIND_BFS
                              else O.dijkstra(g.offsets, g.cols, g.weights, g.n - 1).view(np.int32))
                arcs += g.m
        exp = torch.from_numpy(np.concatenate(expect)).cuda()
        times = -(-(1 << 29) // arcs)
        out, st = lbg.batch_solve(dg, once * times, stats=True)
        assert bool((out.view(times, -1) == exp).all())
        assert (st["atomics"] == 0) == (len(kinds) == 1)


@pytest.mark.parametrize("bound", [BOUND, (1 << 32) - 1])
def test_a_loose_bound_keeps_the_route(bound):
    """The bound sizes the workspace; a batch of few arcs is solved in the
    shared worklist whatever it is."""
    gs = [graphgen.uniform(n=n, k=8, salt=n) for n in (3000, 20000, 100000)]
    u, nb, _ = graphgen.pack(gs)
    dg = lbg.DeviceGraph.from_numpy(u.offsets, u.cols, u.weights)
    queries = [(int(nb[i]), int(nb[i]), int(nb[i + 1]), kind) for i in range(3) for kind in (lbg.KIND_BFS, lbg.KIND_SSSP)]
    ref, s0 = lbg.batch_solve(dg, queries, stats=True)
    got, st = lbg.batch_solve(dg, queries, total_arcs=bound, stats=True)
    assert torch.equal(got, ref)
    assert st["atomics"] > s0["atomics"] // 2 > 0  # one workgroup's atomics are in LDS and not counted
