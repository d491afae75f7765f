"""The searches' queue keys and lists (kappa_refine) where they can go wrong:
32-bit keys with few hash bits (equal keys), the largest weighted degree of
32-bit keys and one more (64-bit keys), pairs at the on-chip capacity and just
above it, areas kept in memory, and the later boundary list past its room."""
import numpy as np
import pytest

import paper_0910_2004_amd as K
from test_gpu_refine import check_refine, say
from workloads import csr_from_edges, grid2d, path_graph, rgg

pytestmark = pytest.mark.gpu


def heavy_edge(g, w):
    """g with the weight of its first edge set so that the weighted degree of
    its first node is w."""
    ew = g.ew.copy()
    x = g.xadj
    v, u = 0, int(g.adj[0])
    rest = int(ew[1:x[1]].sum())
    back = x[u] + int(np.searchsorted(g.adj[x[u]:x[u + 1]], v))
    ew[0] = ew[back] = w - rest
    return type(g)(g.n, g.xadj, g.adj, ew, g.vw)


@pytest.mark.parametrize("wd", [1 << 10, (1 << 16) - 1, 1 << 16, 1 << 20, (1 << 31) - 5])
def test_key_widths(wd):
    # unit weights and one heavy edge: nearly all gains are equal small numbers,
    # told apart by whatever hash bits the heavy edge leaves to the key
    for name, g in (("grid30x31", grid2d(30, 31)), ("rgg5000", rgg(5000, seed=17))):
        h = heavy_edge(g, wd)
        for k in (2, 6):
            part = np.random.default_rng(k + wd % 97).integers(0, k, g.n).astype(np.int32)
            check_refine(h, part, k, "fast", seed=5, what=f"{name} wd={wd} k={k}")
        part = (np.arange(g.n) * 4 // g.n).astype(np.int32)
        check_refine(h, part, 4, "strong", seed=6, what=f"{name} wd={wd} blocks")


@pytest.mark.parametrize("qcap", [0, 500])
def test_wide_keys_in_memory(qcap, monkeypatch):
    monkeypatch.setenv("KAPPA_REFINE_QCAP", str(qcap))
    for wd in (300, (1 << 16) - 1, 1 << 18):
        g = heavy_edge(rgg(3000, seed=4), wd)
        part = np.random.default_rng(1).integers(0, 3, g.n).astype(np.int32)
        check_refine(g, part, 3, "fast", seed=2, what=f"qcap={qcap} wd={wd}")


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097])
def test_pair_sizes(n):
    # one pair of n nodes: group sizes and the on-chip capacity
    g = rgg(n, seed=n) if n > 2 else path_graph([1] * (n - 1))
    part = (np.arange(g.n) % 2).astype(np.int32)
    check_refine(g, part, 2, "fast", seed=n, what=f"alternating n={n}")
    part = (np.arange(g.n) * 10 < g.n).astype(np.int32)   # unbalanced: many kept moves
    check_refine(g, part, 2, "strong", seed=n, what=f"unbalanced n={n}")


def test_later_list_overflow():
    # one block holds nearly everything, so that balancing moves more nodes (and
    # lists more of their neighbours) than the later list has room for
    for rows, cols in ((40, 50), (90, 100)):
        g = grid2d(rows, cols)
        for k in (2, 3):
            part = np.zeros(g.n, np.int32)
            part[: k] = np.arange(k)
            _, st = check_refine(g, part, k, "strong", seed=1, alpha_num=1, alpha_den=1,
                                 what=f"grid {rows}x{cols} k={k}")
            say(f"grid {rows}x{cols} k={k}: kept {st['kept']} of {g.n} nodes")
            assert st["kept"] > g.n // 4


def test_long_rows():
    # hubs (rows read by whole waves, rows of more than one wave in a search)
    n = 3000
    a = np.concatenate([np.zeros(n - 1, np.int64), np.full(n - 2, 1)])
    b = np.concatenate([np.arange(1, n), np.arange(2, n)])
    w = 1 + (np.arange(len(a)) % 7)
    g = csr_from_edges(n, a, b, w.astype(np.uint32))
    for k in (2, 5):
        part = np.random.default_rng(k).integers(0, k, n).astype(np.int32)
        check_refine(g, part, k, "fast", seed=9, what=f"two hubs k={k}")
    assert K.REFINE_K_MAX == 256
