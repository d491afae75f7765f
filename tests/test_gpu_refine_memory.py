"""kappa_refine where the allocator has no room for the pairs' rows (8 bytes per
CSR entry): the searches then read the graph's own rows, with the same result."""
import ctypes

import numpy as np
import pytest

import paper_0910_2004_amd as K
from test_gpu_refine import check_refine, say
from workloads import random_graph, rgg, rmat

pytestmark = pytest.mark.gpu


class Limited:
    """torch's caching allocator, refusing blocks above a limit."""

    def __init__(self, limit):
        self.limit, self.refused = limit, 0

    def __enter__(self):
        import torch
        torch.cuda.synchronize()
        dev = torch.cuda.current_device()

        def alloc(n, stream, ctx):
            if n > self.limit:
                self.refused += 1
                return None
            return torch.cuda.caching_allocator_alloc(int(n), dev, int(stream or 0))

        def free(p, n, stream, ctx):
            torch.cuda.caching_allocator_delete(int(p))

        self.cbs = (K._lib._ALLOC_FN(alloc), K._lib._FREE_FN(free))
        assert K.lib().kappa_set_allocator(self.cbs[0], self.cbs[1], None) == K.OK
        return self

    def __exit__(self, *exc):
        assert K.lib().kappa_set_allocator(K._lib._ALLOC_FN(), K._lib._FREE_FN(), None) == K.OK


@pytest.mark.parametrize("k", [2, 9])
def test_no_room_for_rows(k):
    for name, g, heavy in (("random", random_graph(3000, 90000, seed=4, wmax=30, cmax=6, cmin=0), 0),
                           ("rmat11", rmat(11, 40, seed=4, wseed=5, wmax=20), 0),
                           ("rgg9000", rgg(9000, seed=2, mean_degree=40.0), 0),
                           ("heavy", random_graph(2000, 60000, seed=6, wmax=1 << 22), 1)):
        part = np.random.default_rng(k).integers(0, k, g.n).astype(np.int32)
        rows = 8 * g.nnz
        with Limited(rows) as a:
            say(name, k, "rows of", rows, "bytes refused")
            check_refine(g, part, k, "strong", seed=k, what=f"{name} k={k}")
            check_refine(g, (np.arange(g.n) * k // g.n).astype(np.int32), k, "fast", seed=k,
                         what=f"{name} bands k={k}")
        assert a.refused > 0


def test_no_room_at_all():
    g = rgg(2000, seed=1)
    import torch
    from gpu_util import dev
    d, p = dev(g), torch.zeros(g.n, dtype=torch.int32, device="cuda")
    with Limited(1000) as a:
        with pytest.raises(K.KappaError) as e:
            K.kappa_refine(d, p, 4)
        assert e.value.status == K.E_NOMEM and a.refused > 1
    assert ctypes.c_int(K.kappa_validate(d)).value == K.OK
