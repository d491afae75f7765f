"""HIP-graph replays of kappa_coarsen where a batch of levels ends early: the
levels launched are the same whether the sequence runs directly, is captured or
is replayed."""
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import check_hierarchy, compare_hierarchy, dev
from workloads import csr_from_edges, grid2d, rgg

pytestmark = pytest.mark.gpu


# just above the small form's 4096 nodes (its trial ends the first batch without
# taking the level), below it, and a few levels above it
@pytest.mark.parametrize("name,make", [("grid70x72", lambda: grid2d(70, 72)),
                                       ("grid60x64", lambda: grid2d(60, 64)),
                                       ("rgg9001", lambda: rgg(9001, seed=2)),
                                       ("rgg2^15", lambda: rgg(1 << 15, seed=3))])
@pytest.mark.parametrize("tail", [False, True])
def test_batches_that_end_early(name, make, tail):
    import torch
    g = make()
    dg = dev(g)
    OH = O.coarsen(g, O.EXPANSION_STAR2, 7, 40, 1, 20, 64, round_stats=True)
    part0 = torch.empty(g.n, dtype=torch.int32, device="cuda")
    K.graphs_enable(True)
    K.tail_enable(tail)
    try:
        for rep in range(6):   # direct, capture, replays
            print(name, "tail", tail, "call", rep, flush=True)
            check_hierarchy(g, O.EXPANSION_STAR2, 7, 40, k=2, oracle_h=OH, dg=dg, part0=part0)
            assert int(torch.ones(1 << 16, device="cuda").sum().item()) == 1 << 16
    finally:
        K.tail_enable(False)
        K.graphs_enable(False)


def chains_and_stars(stars):
    """100 chains of ascending weights (a hundred rounds; the level is handed
    back for more) and 1500 light edges from the given number of centres."""
    import numpy as np
    v = np.arange(20000)
    v = v[v % 200 != 199]
    leaf = np.random.default_rng(1).permutation(20000)[:1500]
    a = np.concatenate([v, leaf])
    b = np.concatenate([v + 1, 20000 + np.arange(1500) % stars])
    return csr_from_edges(20005, a, b, np.concatenate([10 + v % 200, np.ones(1500)]).astype(np.uint32))


def test_scratch_of_long_rows():
    # two graphs of one size, handed back at one round, one with a row above
    # 1024 entries: each replays its own sequences
    gs = [chains_and_stars(1), chains_and_stars(5)]
    assert gs[0].nnz == gs[1].nnz and gs[0].degrees().max() > 1024 > gs[1].degrees().max() > 255
    dgs = [dev(g) for g in gs]
    hs = [O.coarsen(g, O.WEIGHT, 7, 3000, 1, 20, 64, round_stats=True) for g in gs]
    assert all(h.levels[0].rounds > 50 for h in hs)
    K.graphs_enable(True)
    try:
        for i in (0, 0, 0, 1, 1, 1, 0, 1):
            print("graph", i, flush=True)
            H, OH = check_hierarchy(gs[i], O.WEIGHT, 7, 3000, k=2, oracle_h=hs[i], dg=dgs[i],
                                    check_rounds=False)
            for l in range(len(H) - 1):   # (slot 64 sums all rounds from 64 on)
                ol = OH.levels[l]
                r, p, d = H.round_stats(l)
                assert r == ol.rounds, f"graph {i} level {l}: rounds"
                assert list(p[:63]) == list(ol.round_active[:r][:63]), f"graph {i} level {l}"
                assert list(d[:63]) == list(ol.round_degree[:r][:63]), f"graph {i} level {l}"
    finally:
        K.graphs_enable(False)


def test_servers_of_their_own():
    # steps of equal sizes on one server after another, interrupts among them:
    # a step watches the flag of its own server
    gs = [grid2d(60, 50), rgg(5001, seed=4)]
    hs = [O.coarsen(g, O.EXPANSION_STAR2, 42, 40, 1, 20, 64) for g in gs]
    dgs = [dev(g) for g in gs]
    K.graphs_enable(True)
    try:
        for rep in range(6):
            srv = K.Server(O.EXPANSION_STAR2, 42)
            ids = [srv.admit(d, 40) for d in dgs]
            done, steps = set(), 0
            srv.interrupt(rep % 2 == 1)   # level by level
            while srv.active():
                done |= set(srv.step())
                steps += 1
            print("server", rep, "steps", steps, flush=True)
            assert done == set(ids)
            for i, h in zip(ids, hs):
                compare_hierarchy(srv.take(i), h, check_rounds=False, k=2)
            del srv
    finally:
        K.graphs_enable(False)
