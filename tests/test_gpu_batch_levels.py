"""Graphs handed out of a batch where a launch's table of levels ends: 15 to 17
and 33 levels, graphs of one level and of no node beside them."""
import numpy as np
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import compare_hierarchy
from workloads import grid2d, path_graph, rgg, star_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [14, 15, 16, 17, 32, 33])
def test_levels(leaves):
    graphs = [star_graph(leaves), path_graph([3]), O.Graph(0, np.zeros(1, np.int64),
              np.zeros(0, np.int32), np.zeros(0, np.uint32), np.zeros(0, np.uint32)),
              rgg(3000, seed=leaves), star_graph(leaves + 20), grid2d(9, 9)]
    u, off = K.DeviceGraph.union(graphs)
    B = K.kappa_coarsen_batch(u, off, K.EXPANSION_STAR2, 7, 1, 1, 1000, 256)
    for g, G in enumerate(graphs):
        OH = O.coarsen(G, K.EXPANSION_STAR2, 7, 1, 1, 1000, 256)
        compare_hierarchy(B.hierarchy(g), OH, check_rounds=False, check_uncoarsen=G.n > 0, k=3)
