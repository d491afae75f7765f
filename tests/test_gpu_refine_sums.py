"""kappa_refine of graphs whose sums of node or edge weights pass 2^32 - 1:
block weights, cuts and gains are then kept in 64 bits, and the result is the
oracle's as on any other graph."""
import numpy as np
import pytest

from test_gpu_refine import check_refine, say
from workloads import csr_from_edges, grid2d, rgg

pytestmark = pytest.mark.gpu


def weighted(g, wlo, whi, clo, chi, seed):
    """g with edge weights in [wlo, whi] and node weights in [clo, chi]."""
    rng = np.random.default_rng(seed)
    src = np.repeat(np.arange(g.n, dtype=np.int64), np.diff(g.xadj))
    up = src < g.adj
    w = rng.integers(wlo, whi, int(up.sum()), endpoint=True).astype(np.uint32)
    c = rng.integers(clo, chi, g.n, endpoint=True).astype(np.uint32)
    return csr_from_edges(g.n, src[up], g.adj[up], w, c)


def parts(n, k, seed):
    rng = np.random.default_rng(seed)
    yield "random", rng.integers(0, k, n).astype(np.int32)
    yield "bands", (np.arange(n) * k // n).astype(np.int32)
    yield "uneven", np.where(rng.random(n) < 0.7, 0, rng.integers(0, k, n)).astype(np.int32)


def check(g, k, preset, what):
    for kind, part in parts(g.n, k, k):
        say(what, kind, k, preset)
        check_refine(g, part, k, preset, seed=3, what=f"{what} {kind} k={k}")


GRAPHS = [("grid30x31", lambda: grid2d(30, 31)), ("rgg5000", lambda: rgg(5000, seed=2))]


@pytest.mark.parametrize("k", [2, 7])
@pytest.mark.parametrize("name,make", GRAPHS)
def test_node_weights(name, make, k):
    # c(V) above 2^32, single blocks above and below it
    for lo, hi in ((1 << 30, (1 << 32) - 1), (1 << 21, 1 << 22)):
        check(weighted(make(), 1, 9, lo, hi, 5), k, "fast", f"{name} c to {hi}")


@pytest.mark.parametrize("qcap", [None, 0, 400])
@pytest.mark.parametrize("k", [2, 7])
@pytest.mark.parametrize("name,make", GRAPHS)
def test_edge_weights(name, make, k, qcap, monkeypatch):
    # cuts above 2^32; weighted degrees above it as well, with up to a few
    # hundred nodes of one gain
    if qcap is not None:
        monkeypatch.setenv("KAPPA_REFINE_QCAP", str(qcap))
    for lo, hi in ((1 << 31, (1 << 32) - 1), ((1 << 32) - 1, (1 << 32) - 1), (1 << 22, 1 << 23)):
        check(weighted(make(), lo, hi, 1, 3, 6), k, "strong", f"{name} w to {hi}")


def test_long_rows_of_heavy_edges():
    # a star and a path: a weighted degree of 2^43
    n = 3000
    a = np.concatenate([np.zeros(n - 1, np.int64), np.arange(1, n - 1)])
    b = np.concatenate([np.arange(1, n), np.arange(2, n)])
    w = np.full(len(a), (1 << 32) - 1, np.uint32)
    w[::3] = 1
    g = csr_from_edges(n, a, b, w, np.full(n, (1 << 32) - 1, np.uint32))
    check(g, 3, "fast", "star and path")
