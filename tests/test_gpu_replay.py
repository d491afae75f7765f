"""HIP-graph replays of kappa_coarsen where a batch of levels ends early: the
levels launched are the same whether the sequence runs directly, is captured or
is replayed."""
import pytest

import oracle as O
import paper_0910_2004_amd as K
from gpu_util import check_hierarchy, dev
from workloads import grid2d, rgg

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
