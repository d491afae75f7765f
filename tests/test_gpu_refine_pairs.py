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


# block 0 in a small pair; small and large pairs in turn
SIZES8 = (1, 1.2, 4, 4.5, 1.1, 0.9, 5, 3)


@pytest.mark.parametrize("eps", [(3, 100), (4, 1)])
@pytest.mark.parametrize("k,qcap", [(8, 900), (64, 150)])
def test_small_and_large_pairs_side_by_side(k, qcap, eps, monkeypatch):
    # a lowered on-chip capacity between the sizes of the small and the large
    # pairs of a colour; eps 4 leaves the blocks as uneven as they are
    monkeypatch.setenv("KAPPA_REFINE_QCAP", str(qcap))
    sizes = SIZES8 * (k // 8)
    for name, g in (("grid70x80", grid2d(70, 80)), ("rgg6001", rgg(6001, seed=8))):
        for part in (uneven_random(g.n, sizes, k), uneven_bands(g.n, sizes)):
            for preset in ("fast", "strong"):
                say(name, k, preset)
                check_refine(g, part, k, preset, seed=k, eps=eps, what=f"{name} k={k} {preset}")


@pytest.mark.parametrize("eps", [(3, 100), (4, 1)])
def test_pairs_on_both_sides_of_the_capacity(eps):
    # the kernel's own capacity, 4096 nodes: pairs of about 2600 and 11000 nodes
    for name, g in (("grid150x160", grid2d(150, 160)), ("rgg25001", rgg(25001, seed=3))):
        for part in (uneven_random(g.n, SIZES8, 4), uneven_bands(g.n, SIZES8)):
            say(name)
            _, st = check_refine(g, part, 8, "strong", seed=2, eps=eps, what=name)
            assert st["adoptions"] > 0


def test_uneven_64():
    # 64 blocks: small pairs of 400 nodes beside pairs of 7000 and more
    g = rgg(1 << 17, seed=6)
    sizes = [1 if i % 4 < 2 else 19 for i in range(64)]
    for part in (uneven_bands(g.n, sizes), uneven_random(g.n, sizes, 1)):
        check_refine(g, part, 64, "minimal", seed=4, eps=(1, 1), what="uneven k=64")
