"""SSSP levels around the sizes at which a level's workgroups change from half
of the resident ones to all of them (tiles of 512 arcs, 4 for each of the
wavefronts that take part), against the oracle, bit for bit."""
import numpy as np
import pytest

import graphgen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)
from paper_1711_00231_amd import lbg  # noqa: E402

O = oracle.get()
FEW = 4096 // 2 * 4 * 512  # arcs up to which half of 4,096 resident wavefronts take part


@pytest.fixture(autouse=True)
def _reset():
    yield
    lbg.set_addressing(0)


@pytest.mark.parametrize("arcs", [FEW // 4 + 1, FEW - 1, FEW + 1, FEW + FEW // 3, 2 * FEW + 513])
def test_level_of(arcs):
    """The source's second level has exactly `arcs` arcs (a graph with more
    than 16 arcs per node, so nothing is deferred)."""
    deg = 48
    k = arcs // deg
    pool = k // 2
    rng = np.random.default_rng(arcs % 1009)
    last = arcs - k * deg
    src = np.concatenate([np.zeros(k + 1, np.int64), np.repeat(1 + np.arange(k), deg), np.full(last, k + 1)])
    dst = np.concatenate([1 + np.arange(k + 1), k + 2 + rng.integers(0, pool, arcs)])
    w = np.concatenate([rng.integers(1, 100, k + 1), rng.integers(1, 100, arcs)])
    n = k + 2 + pool
    order = np.argsort(src, kind="stable")
    offsets = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int32)
    cols, wts = dst[order].astype(np.int32), w[order].astype(np.uint32)
    assert cols.size > 16 * n
    exp = O.dijkstra(offsets, cols, wts, 0)
    dg = lbg.DeviceGraph.from_numpy(offsets, cols, wts)
    for kw in ({}, {"packed": True}, {"ordered": True}):
        for wide in (0, 1):
            lbg.set_addressing(wide)
            d = lbg.sssp(dg, 0, **kw).cpu().numpy().view(np.uint32)
            assert np.array_equal(d, exp), (arcs, kw, wide)
