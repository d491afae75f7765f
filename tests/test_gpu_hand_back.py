"""Matchings the finisher hands back to the grid for the entries of their
pending rows: at, below and above that limit, with rows short, of the wave class
and in chunks, and through the single-step matcher."""
import numpy as np
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import check_hierarchy, dev
from workloads import csr_from_edges, random_graph, rmat

pytestmark = pytest.mark.gpu


def chained(hubs, leaves, seed):
    """Rows of `leaves` and more entries whose best edges form a chain, so that
    each round matches few of them."""
    rng = np.random.default_rng(seed)
    a = np.repeat(np.arange(hubs, dtype=np.int64), leaves)
    b = hubs + (np.tile(np.arange(leaves), hubs) * 7 + a * 3) % (leaves * 2)
    h = np.arange(hubs - 1)
    w = np.concatenate([rng.integers(1, 9, len(a)), 1000 + h * 3])
    return csr_from_edges(hubs + 2 * leaves, np.concatenate([a, h]), np.concatenate([b, h + 1]),
                          w.astype(np.uint32))


@pytest.mark.parametrize("rating", [0, 2, 4])
@pytest.mark.parametrize("make", [lambda: chained(300, 100, 1), lambda: chained(330, 100, 2),
                                  lambda: chained(60, 1100, 3), lambda: random_graph(4000, 90000, seed=1, wmax=3),
                                  lambda: random_graph(12000, 300000, seed=2, wmax=1000),
                                  lambda: rmat(13, 24, seed=3, wseed=4)])
def test_hand_back(make, rating):
    g = make()
    # (a level of more than 64 rounds sums the rest in the last slot)
    check_hierarchy(g, rating, 6, 50, k=4, check_rounds=False)
    mate, rounds, matched = K.kappa_match(dev(g), rating, 77)
    want, wmatched, wrounds = O.match_rounds(g, rating, 77)[:3]
    assert np.array_equal(mate.cpu().numpy(), want)
    assert (matched, rounds) == (wmatched, wrounds)
