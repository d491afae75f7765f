"""The way back up over many levels per launch, and the cut of one level,
where they can go wrong: more levels than a launch's table holds, one level,
sizes around the blocks and tiles, several groups of levels, tiles with more
empty rows than are staged, arrays that are not aligned to 16 bytes."""
import numpy as np
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import check_hierarchy, dev
from workloads import csr_from_edges, grid2d, path_graph, rgg, rmat, star_graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("leaves", [1, 22, 23, 24, 25, 47, 70])
def test_many_levels(leaves):
    # a star loses one node a level
    for k in (1, 3, 4096):
        H, _ = check_hierarchy(star_graph(leaves), 2, 9, 1, stall=(1, 1000), max_levels=256, k=k,
                               check_rounds=False)
        assert len(H) == leaves + 1


@pytest.mark.parametrize("g", [path_graph([1]), path_graph(list(range(1, 256))), grid2d(32, 32),
                               grid2d(31, 33), rgg(4097, seed=3), rmat(12, 16, seed=2)],
                         ids=lambda g: f"n{g.n}")
def test_sizes(g):
    for k in (2, 64, 1000):
        check_hierarchy(g, 4, 3, 2, k=k, check_rounds=False, part_seed=k)


def test_several_groups():
    g = rgg(1 << 20, seed=5)   # 9 M maps to follow over all levels
    check_hierarchy(g, 1, 3, 64, k=64, check_rounds=False)


def sparse_rows(n, step):
    v = np.arange(0, n - step, step, dtype=np.int64)
    return csr_from_edges(n, v, v + step, (1 + v % 7).astype(np.uint32),
                          (1 + np.arange(n) % 3).astype(np.uint32))


@pytest.mark.parametrize("n,step", [(5000, 1), (9000, 4096), (300000, 7), (2000000, 900)])
def test_empty_rows(n, step):
    check_cut(sparse_rows(n, step), 5, 0)


@pytest.mark.parametrize("off", [0, 1, 2, 3])
def test_alignment(off):
    for g in (rgg(3001, seed=1), rmat(13, 8, seed=4)):
        check_cut(g, 7, off)


def check_cut(g, k, off):
    import torch
    dg = dev(g)
    part = ((np.arange(g.n, dtype=np.int64) * 2654435761 >> 7) % k).astype(np.int32)

    def moved(t):   # the same values, off elements into a buffer
        b = torch.zeros(t.numel() + off + 4, dtype=t.dtype, device=t.device)
        b[off:off + t.numel()] = t
        return b[off:off + t.numel()]
    dg.adj, dg.ew = moved(dg.adj), moved(dg.ew)
    want = O.cut_balance(g, part, k, 3, 100)
    p = torch.from_numpy(part).cuda()
    res, bw = K.kappa_cut_balance(dg, p, k, 3, 100)[:2]
    assert res.as_tuple() == want.as_tuple()
    assert np.array_equal(np.bincount(part, weights=g.vw, minlength=k).astype(np.int64),
                          bw.cpu().numpy().astype(np.int64))
