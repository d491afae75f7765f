"""Contraction of short rows (kappa_contract): merged rows of up to one entry a
lane (16) and just above it in one wave, rows whose entries nearly all repeat,
rows of one pair's own edge, and empty rows, against the oracle."""
import numpy as np
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import assert_graph_equal, dev, graph_np
from workloads import (complete_graph, csr_from_edges, cycle_graph, grid2d, path_graph, random_graph,
                       rgg)

pytestmark = pytest.mark.gpu


def ladders(count, d, seed):
    """`count` pairs of nodes, both joined to the same d of `count` further nodes
    that are matched among themselves: merged rows of 2 d entries, each key up
    to four times."""
    rng = np.random.default_rng(seed)
    a, b = [], []
    for i in range(count):
        to = rng.choice(count // 2, d // 2, replace=False) * 2
        to = np.concatenate([to, to + 1])[:d]
        for v in (2 * i, 2 * i + 1):
            a.append(np.full(len(to), v))
            b.append(2 * count + to)
    a, b = np.concatenate(a + [np.arange(count) * 2]), np.concatenate(b + [np.arange(count) * 2 + 1])
    g = csr_from_edges(3 * count, a, b, rng.integers(1, 1000, len(a)).astype(np.uint32))
    mate = np.full(g.n, -1, np.int32)
    mate[0:2 * count:2], mate[1:2 * count:2] = np.arange(1, 2 * count, 2), np.arange(0, 2 * count, 2)
    return g, mate


def check(g, mate):
    import torch
    cmap, cg = K.kappa_contract(dev(g), torch.from_numpy(mate).cuda())
    ocmap, og = O.contract(g, mate)[:2]
    assert np.array_equal(cmap.cpu().numpy()[:g.n], ocmap)
    assert_graph_equal(graph_np(cg), og)


@pytest.mark.parametrize("d", [2, 4, 6, 8, 10, 16])
def test_repeated_entries(d):
    for count in (64, 129, 1000):
        check(*ladders(count, d, d))


@pytest.mark.parametrize("n", [2, 3, 8, 9, 10, 17, 18])
def test_complete(n):
    # merged rows of 2 (n - 1) - 2 entries and, unmatched, of n - 1
    g = complete_graph(n)
    for pairs in (0, 1, n // 2):
        mate = np.full(n, -1, np.int32)
        v = np.arange(2 * pairs)
        mate[:2 * pairs] = v ^ 1
        check(g, mate)


@pytest.mark.parametrize("name,g", [("path", path_graph([3, 1, 4, 1, 5] * 300)), ("cycle", cycle_graph(1025)),
                                    ("grid", grid2d(37, 41)), ("rgg", rgg(3000, seed=3)),
                                    ("sparse", random_graph(2000, 2500, seed=1, wmax=9)),
                                    ("mixed", random_graph(2000, 8000, seed=2, wmax=9)),
                                    ("edgeless", csr_from_edges(100, np.zeros(0, np.int64), np.zeros(0, np.int64)))])
def test_matched(name, g):
    for rating in (0, 2):
        check(g, O.match_rounds(g, rating, 5)[0])
    check(g, np.full(g.n, -1, np.int32))
