"""The bisection order and the renumbering where their paths meet: sizes around
the points a block keeps on chip and its tiles, crowded coordinates (runs of
equal short keys, in order and not, longer than are put in order by a thread),
equal coordinates, infinities, and rows of 15 .. 17, 63 .. 65 and more entries.
Sorts around one tile."""
import numpy as np
import pytest

import paper_0910_2004_amd as K
from gpu_util import dev, graph_np, assert_graph_equal
from oracle.rcb import rcb_order, relabel
from test_gpu_relabel import dev_order
from workloads import complete_graph, csr_from_edges, rgg, rmat

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 511, 4095, 4096, 4097, 8191, 8192, 8193, 12289,
                               16385, 100003])
@pytest.mark.parametrize("leaf", [1, 2, 31, 4096, 6000])
def test_sizes(n, leaf):
    pts = np.random.default_rng(n).random((n, 2))
    assert np.array_equal(dev_order(pts, leaf), rcb_order(pts, leaf))


def crowded(kind, n, rng):
    if kind == "outlier":      # all but one in a few short keys, out of order
        p = 1.0 + rng.random((n, 2)) * 2.0 ** -40
        p[n // 2] = -1e300
    elif kind == "outlier_x":
        p = rng.random((n, 2))
        p[:, 0] = 1.0 + p[:, 0] * 2.0 ** -45
        p[1, 0] = 1e300
    elif kind == "outlier_y":
        p = rng.random((n, 2))
        p[:, 1] = 1.0 + p[:, 1] * 2.0 ** -45
        p[1, 1] = 1e300
    elif kind == "equal":
        p = np.ones((n, 2))
    elif kind == "columns":    # long runs of equal x
        p = np.stack([rng.integers(0, 7, n), rng.random(n)], -1)
    elif kind == "lattice":
        p = rng.integers(-9, 9, (n, 2)).astype(np.float64)
    elif kind == "pairs":      # short runs, equal and not
        p = np.repeat(rng.random(((n + 2) // 3, 2)), 3, axis=0)[:n]
        p[::3] = np.nextafter(p[::3], 2.0)
        p = p[rng.permutation(n)]
        p[0] = -1.0
    else:                      # infinities and both zeros
        p = rng.normal(size=(n, 2))
        p[::5] = np.inf
        p[1::7] = -np.inf
        p[2::11] = -0.0
        p[3::11] = 0.0
    return p


@pytest.mark.parametrize("kind", ["outlier", "outlier_x", "outlier_y", "equal", "columns", "lattice",
                                  "pairs", "inf"])
def test_crowded(kind):
    for n in (40, 5000, 20011):
        pts = crowded(kind, n, np.random.default_rng(n))
        for leaf in (1, 32):
            assert np.array_equal(dev_order(pts, leaf), rcb_order(pts, leaf)), (n, leaf)


@pytest.mark.parametrize("size", [15, 16, 17, 18, 63, 64, 65, 66, 200])
def test_row_lengths(size):
    # a clique of rows of size - 1 entries, paths and isolated nodes beside it
    import torch
    a, b = np.triu_indices(size, 1)
    q = size + np.arange(300)
    g = csr_from_edges(size + 340, np.concatenate([a, q]), np.concatenate([b, q + 1]),
                       (1 + np.arange(len(a) + 300) % 11).astype(np.uint32))
    perm = np.random.default_rng(size).permutation(g.n).astype(np.int32)
    got = graph_np(K.kappa_relabel(dev(g), torch.from_numpy(perm).cuda()))
    assert_graph_equal(got, relabel(g, perm))


@pytest.mark.parametrize("make", [lambda: rmat(14, 16, seed=3, wseed=1), lambda: rgg(50001, seed=2),
                                  lambda: complete_graph(129)])
def test_mixed_rows(make):
    import torch
    g = make()
    perm = np.random.default_rng(1).permutation(g.n).astype(np.int32)
    got = graph_np(K.kappa_relabel(dev(g), torch.from_numpy(perm).cuda()))
    assert_graph_equal(got, relabel(g, perm))


def test_row_of_more_than_24_bits():
    # the offsets' scan adds values past 2^24 in 64 bits
    import torch
    from workloads import star_graph
    g = star_graph((1 << 24) + 5)
    perm = ((np.arange(g.n, dtype=np.int64) * 5 + 3) % g.n).astype(np.int32)
    assert g.n % 5
    got = graph_np(K.kappa_relabel(dev(g), torch.from_numpy(perm).cuda()))
    assert_graph_equal(got, relabel(g, perm))
