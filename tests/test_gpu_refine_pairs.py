"""kappa_refine where the pairs of one colour run side by side and see each
other's work: the later boundary list, which all pairs of a launch append to
while each walks it."""
import numpy as np
import pytest

from test_gpu_refine import check_refine, say
from workloads import grid2d, rgg

pytestmark = pytest.mark.gpu


def uneven_random(n, sizes, seed):
    """Blocks of about these relative sizes, nodes at random: every node is
    next to other blocks."""
    p = np.asarray(sizes, float)
    return np.random.default_rng(seed).choice(len(p), n, p=p / p.sum()).astype(np.int32)


def uneven_bands(n, sizes):
    """Runs of consecutive ids of these relative sizes."""
    edge = np.rint(np.cumsum(sizes) / np.sum(sizes) * n).astype(np.int64)
    return np.searchsorted(edge, np.arange(n), side="right").astype(np.int32)


@pytest.mark.parametrize("k", [8, 32])
def test_large_pairs_side_by_side(k, monkeypatch):
    # every pair above the on-chip capacity, several to a colour, each with
    # many adoptions: the list grows over several tiles, and past its room,
    # while the other pairs of the colour read it
    monkeypatch.setenv("KAPPA_REFINE_QCAP", "64")
    for name, g in (("grid120x130", grid2d(120, 130)), ("rgg20001", rgg(20001, seed=3))):
        for part in (uneven_random(g.n, [1 + i % 3 for i in range(k)], k),
                     uneven_bands(g.n, [1 + i % 3 for i in range(k)])):
            for preset in ("fast", "strong"):
                say(name, k, preset)
                _, st = check_refine(g, part, k, preset, seed=k, what=f"{name} k={k} {preset}")
                assert st["adoptions"] > 0
