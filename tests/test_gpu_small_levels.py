"""Levels that run whole in one workgroup (n <= 4096, entries + n <= 20480, rows
of at most 255 entries) where its limits and classes lie: sizes at and past each
limit, rows of the wave class, merged rows past a group's, many rounds, empty and
edgeless graphs, weights whose products need 128 bits, stop and stall rules, and
a graph that grows a long row on a coarser level."""
import numpy as np
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import check_hierarchy, dev
from workloads import (complete_graph, csr_from_edges, cycle_graph, grid2d, path_graph, random_graph,
                       rgg, rmat, star_graph)

pytestmark = pytest.mark.gpu
RATINGS = [0, 1, 2, 3, 4]


def circulant(n, d, seed=None):
    """n nodes, each joined to the next d; weights 1, or random with a seed."""
    v = np.repeat(np.arange(n, dtype=np.int64), d)
    u = (v + np.tile(np.arange(1, d + 1), n)) % n
    rng = np.random.default_rng(seed)
    w = np.ones(len(v), np.uint32) if seed is None else rng.integers(1, 50, len(v)).astype(np.uint32)
    return csr_from_edges(n, v, u, w)


@pytest.mark.parametrize("rating", RATINGS)
@pytest.mark.parametrize("g", [path_graph([1]), grid2d(5, 7), grid2d(64, 64), grid2d(63, 65),
                               cycle_graph(4096), cycle_graph(4097), random_graph(4095, 8000, seed=3),
                               random_graph(500, 9990, seed=4, wmax=9, cmax=4, cmin=0),
                               rgg(2200, seed=8), rmat(9, 12, seed=5, wseed=6)],
                         ids=lambda g: f"n{g.n}e{int(g.xadj[-1])}")
def test_ratings(g, rating):
    check_hierarchy(g, rating, 42, 2, k=3)


@pytest.mark.parametrize("n,d", [(4096, 2), (2048, 4), (2276, 4), (2275, 4), (120, 60), (160, 63),
                                 (256, 39), (300, 33), (1000, 9), (2, 1), (3, 1)])
def test_entry_limits(n, d):
    # nnz + n = n (2 d + 1): 2276 * 9 = 20484 is past the limit
    for seed in (None, 7):
        d_ = min(d, (n - 1) // 2) or 1
        check_hierarchy(circulant(n, d_, seed) if n > 2 else path_graph([5]), 4, 3, 2, k=2)


@pytest.mark.parametrize("leaves", [31, 32, 33, 63, 64, 65, 254, 255, 256, 600])
def test_long_rows(leaves):
    check_hierarchy(star_graph(leaves), 2, 9, 1, stall=(1, 1000), max_levels=100, k=2)
    check_hierarchy(complete_graph(min(leaves, 142)), 0, 5, 1, k=2)


@pytest.mark.parametrize("k", [20, 100, 200])
def test_rows_grow(k):
    # hubs of k leaves on a path, each leaf joined to two hubs: the hubs' rows
    # merge into longer ones level by level
    hubs, rng = 12, np.random.default_rng(k)
    e = np.unique(np.repeat(np.arange(hubs), k) * 1000 + rng.integers(0, 900, hubs * k))
    g = csr_from_edges(hubs + 900, np.concatenate([e // 1000, np.arange(hubs - 1)]),
                       np.concatenate([hubs + e % 1000, np.arange(1, hubs)]),
                       np.concatenate([rng.integers(1, 5, len(e)), np.full(hubs - 1, 60)]).astype(np.uint32))
    for rating in (0, 4):
        check_hierarchy(g, rating, 5, 2, stall=(0, 1), k=2)


def test_many_rounds_and_wide_products():
    g = path_graph(list(range(1, 4090)))   # a chain of 2045 rounds; slot 64 sums those from 64 on
    H, _ = check_hierarchy(g, 0, 1, 2, k=2, check_rounds=False)
    K.tail_enable(True)   # the same rounds over global memory
    try:
        T, _ = check_hierarchy(g, 0, 1, 2, k=2, check_rounds=False)
    finally:
        K.tail_enable(False)
    for l in range(len(H) - 1):
        for a, b in zip(H.round_stats(l), T.round_stats(l)):
            assert np.array_equal(a, b), f"level {l}"
    g = random_graph(900, 3000, seed=6, wmax=1000000, cmax=60000)
    for rating in (1, 3, 4):
        check_hierarchy(g, rating, 7, 2, k=2)


def test_stops():
    g = rgg(2000, seed=3)
    for stop_n, stall, levels in ((2000, (1, 20), 64), (1999, (1, 20), 64), (50, (1, 2), 64),
                                  (2, (1, 20), 1), (2, (1, 20), 3), (2, (0, 1), 64)):
        check_hierarchy(g, 4, 3, stop_n, stall=stall, max_levels=levels, k=2)
    iso = csr_from_edges(700, np.zeros(0, np.int64), np.zeros(0, np.int64))
    check_hierarchy(iso, 4, 3, 2, k=2)


@pytest.mark.parametrize("rating", [1, 4])
def test_after_grid_levels(rating):
    for g in (rgg(30000, seed=2), grid2d(150, 149), random_graph(9000, 20000, seed=1)):
        check_hierarchy(g, rating, 11, 16, k=4)


def test_arena_grows():
    g = grid2d(60, 60)
    K.arena_first(100000)
    try:
        check_hierarchy(g, 4, 42, 2, k=3)
    finally:
        K.arena_first(0)


@pytest.mark.parametrize("stop_n,levels", [(4500, 64), (5001, 64), (2, 1), (2, 0), (2, 2)])
def test_stops_at_a_level_that_does_not_fit(stop_n, levels):
    # by nodes (level 0) and by entries (level 1 of the geometric graph)
    for g in (rgg(5001, seed=1), circulant(5001, 3, 2)):
        check_hierarchy(g, 0, 42, stop_n, max_levels=levels, k=2)
    # by a row that grew too long
    hubs, k, rng = 12, 200, np.random.default_rng(3)
    e = np.unique(np.repeat(np.arange(hubs), k) * 1000 + rng.integers(0, 900, hubs * k))
    g = csr_from_edges(hubs + 900, np.concatenate([e // 1000, np.arange(hubs - 1)]),
                       np.concatenate([hubs + e % 1000, np.arange(1, hubs)]),
                       np.concatenate([rng.integers(1, 5, len(e)), np.full(hubs - 1, 60)]).astype(np.uint32))
    check_hierarchy(g, 4, 5, min(stop_n, 900), stall=(0, 1), max_levels=levels, k=2)
