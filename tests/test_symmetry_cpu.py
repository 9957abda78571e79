"""The symmetry check of BFS pull levels on the host: the exactness of its
field arithmetic, sets of one-way arcs whose hash sums used to cancel, and the
kernel itself (tests/c/emul)."""
import ctypes
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

import graphgen

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_00231_amd", "csrc")
P = 2**51 - 129
CXX = ["g++", "-std=c++20", "-w", "-I", CSRC]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    so = str(tmp_path_factory.mktemp("sym") / "libsym.so")
    subprocess.run(CXX + ["-O2", "-ffp-contract=off", "-shared", "-fPIC",
                          os.path.join(ROOT, "tests", "c", "sym_check.cpp"), "-o", so], check=True)
    l = ctypes.CDLL(so)
    vp, i64 = ctypes.c_void_p, ctypes.c_int64
    l.sc_mul.restype = l.sc_small.restype = ctypes.c_double
    l.sc_mul.argtypes = [ctypes.c_double] * 2
    l.sc_small.argtypes = [ctypes.c_double]
    l.sc_products.argtypes = [vp, vp, i64, vp, vp]
    l.sc_passes.argtypes = [vp, vp, i64, i64, ctypes.c_uint64, vp]
    return l


def test_products_are_exact(lib):
    rng = random.Random(1)
    big = [2 * P - 1, -2 * P + 1, P, P - 1, P + 1, 2**51, 1, 0, -1, 3, 2**50 + 1]
    small = [P - 1, 1 - P, 2**50, -(2**50), 2**26 + 1, 1, 0, -1, 7]
    pairs = [(a, b) for a in big for b in small]
    pairs += [(rng.randint(1 - 2 * P, 2 * P - 1), rng.randint(1 - P, P - 1)) for _ in range(20000)]
    for a, b in pairs:
        r = lib.sc_mul(float(a), float(b))
        assert r == int(r) and abs(r) < 2 * P and (int(r) - a * b) % P == 0, (a, b)
        s = lib.sc_small(float(a))
        assert s == int(s) and abs(s) < P and (int(s) - a) % P == 0, a


def _products(lib, u, v, x):
    u, v, x = np.array(u, np.uint32), np.array(v, np.uint32), np.array(x, np.uint64)
    out = np.zeros(4, np.uint64)
    lib.sc_products(u.ctypes.data, v.ctypes.data, u.size, x.ctypes.data, out.ctypes.data)
    return [int(y) for y in out]


@pytest.mark.parametrize("ids", [3, 1000, 2**25])
def test_products_equal_integers(lib, ids):
    rng = random.Random(ids)
    u, v = [], []
    while len(u) < 500:
        a, b = rng.randrange(ids), rng.randrange(ids)
        if a != b:
            u.append(a)
            v.append(b)
    for x in ([0, 1], [P - 1, 5], [rng.randrange(P) for _ in range(2)]):
        exp = []
        for t in x:
            for down in (False, True):
                r = 1
                for a, b in zip(u, v):
                    if (a > b) == down:
                        r = r * (t - (min(a, b) * 2**25 + max(a, b))) % P
                exp.append(r)
        assert _products(lib, u, v, x) == exp
    # and the other way round, in another order: symmetric
    both = list(zip(u + v, v + u))
    rng.shuffle(both)
    out = _products(lib, [a for a, _ in both], [b for _, b in both], [rng.randrange(P) for _ in range(2)])
    assert out[::2] == out[1::2]


def _cycle(a, a2, b, b2):
    return [(a, b), (b, a2), (a2, b2), (b2, a)]


# one-way arcs, whose sums of hash values with a key that was only xored in
# were zero for 2^-19 to 2^-28 of the keys
STRUCTURED = [
    [(3, 2**23 + 12345), (2**23 + 12345, 3 ^ 2**21), (2**23 + 12345, 3 ^ 2**22), (3 ^ 2**21 ^ 2**22, 2**23 + 12345)],
    [(3, 2**19 + 123), (2**19 + 123, 3 ^ 2**17), (2**19 + 123, 3 ^ 2**18), (3 ^ 2**17 ^ 2**18, 2**19 + 123)],
    _cycle(5, 5 ^ 2**22, 2**23 + 9, (2**23 + 9) ^ 2**21),
    _cycle(5, 5 ^ 2**20, 2**21 + 9, (2**21 + 9) ^ 2**19),
    _cycle(0, 1, 2, 3),
    [((v if bin(k).count("1") % 2 else w), (w if bin(k).count("1") % 2 else v))
     for k in range(8) for v, w in [(1 + (k & 1) * 2**18, 2**22 + (k >> 1 & 1) * 2**19 + (k >> 2) * 2**20)]],
]


@pytest.mark.parametrize("case", range(len(STRUCTURED)))
def test_structured_one_way_arcs_never_pass(lib, case):
    """At most 8 points of 2^51 are wrong for 8 arcs: no draw of a million
    passes, not even at one point."""
    u, v = (np.array(x, np.uint32) for x in zip(*STRUCTURED[case]))
    out = np.zeros(2, np.int64)
    lib.sc_passes(u.ctypes.data, v.ctypes.data, u.size, 1_000_000, case, out.ctypes.data)
    assert out.tolist() == [0, 0]


@pytest.fixture(scope="module")
def kernel(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("symrun")
    exe = str(d / "sym_run")
    subprocess.run(CXX + ["-O1", "-ffp-contract=off", "-pthread", "-I", os.path.join(ROOT, "tests", "c", "emul"),
                          os.path.join(ROOT, "tests", "c", "emul", "sym_run.cpp"), "-o", exe], check=True)

    def run(n, src, dst, blocks):
        g = graphgen.from_edges(n, np.array(src), np.array(dst), None, "g")
        with open(d / "g", "wb") as f:
            np.array([g.n, g.m], dtype=np.int32).tofile(f)
            np.asarray(g.offsets, dtype=np.int32).tofile(f)
            np.asarray(g.cols, dtype=np.int32).tofile(f)
        rng = random.Random(blocks)
        r = subprocess.run([exe, str(d / "g"), str(blocks)] + [str(rng.randrange(P)) for _ in range(2)],
                           capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-300:]
        return r.stdout.strip() == "1"

    return run


@pytest.mark.parametrize("blocks", [1, 3, 8])
@pytest.mark.parametrize("half", [1, 700, 9000])
def test_kernel(kernel, blocks, half):
    rng = np.random.default_rng(half)
    n = 1000
    u = (rng.random(half) ** 2 * n).astype(int)
    v = rng.integers(0, n, half)
    loops = rng.integers(0, n, 5)
    s, d = np.concatenate([u, v, loops]), np.concatenate([v, u, loops])
    assert kernel(n, s, d, blocks)
    k = int(np.nonzero(u != v)[0][-1])
    drop = np.arange(s.size) != k
    assert not kernel(n, s[drop], d[drop], blocks)
    one_way = STRUCTURED[4]
    assert not kernel(n, np.append(s, [a for a, _ in one_way]), np.append(d, [b for _, b in one_way]), blocks)


@pytest.mark.parametrize("degree", [4, 31, 33, 100, 600])
def test_sample(kernel, degree):
    """The sample turns down a digraph of any degree up to its longest lists,
    and no symmetric graph."""
    rng = np.random.default_rng(degree)
    n = 5000
    u, v = np.repeat(np.arange(n), degree), rng.integers(0, n, n * degree)
    assert not kernel(n, u, v, 0)
    u, v = u[: u.size // 2], v[: v.size // 2]
    assert kernel(n, np.concatenate([u, v]), np.concatenate([v, u]), 0)
