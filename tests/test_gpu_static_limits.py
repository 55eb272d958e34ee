"""GPU: the allocation-free solve near the size of its scratch array, and with fewer colour bitmaps
than a solve with buffers of its own: what it accepts equals the plain solve."""
from fractions import Fraction as F

import numpy as np
import pytest

from paper_2608_03695_amd import gen

pytestmark = pytest.mark.gpu


def _same(g, **kw):
    m, r = g.leiden(**kw)
    ms, rs = g.leiden(no_alloc=True, **kw)
    assert np.array_equal(m, ms)
    assert np.array_equal(r["q_components"], rs["q_components"])
    for k in ("sweeps", "moves", "refine_rounds", "merges", "levels_run", "n_communities"):
        assert r[k] == rs[k], k


@pytest.mark.parametrize("n,edges", [(694_032, 10), (650_000, 3000)])
def test_few_entries_and_one_starting_community_fit(n, edges):
    """Nearly every unit is one of the next level: its buffers are as large as level 0's."""
    from paper_2608_03695_amd import mslm
    tg = gen.from_edge_lists(n, [[(2 * i, 2 * i + 1) for i in range(edges)]], name="few")
    g = mslm.Graph(tg, 1)
    _same(g, gamma=F(1), initial=np.zeros(n, np.int32))
    g.close()


@pytest.mark.parametrize("gamma", [F(1), F(40)], ids=["coarse", "fine"])
def test_more_colours_than_bitmaps(gamma):
    """Cliques of 70 and one of 150: levels with more than 64 colours, among them levels of nearly
    as many units as level 0 has (at the finer resolution)."""
    from paper_2608_03695_amd import mslm
    rng = np.random.default_rng(3)
    slices = []
    for _ in range(4):
        perm = rng.permutation(570)
        sizes = [150] + [70] * 6
        edges, at = [], 0
        for size in sizes:
            edges += [(int(perm[at + i]), int(perm[at + j])) for i in range(size) for j in range(i)]
            at += size
        slices.append(edges)
    g = mslm.Graph(gen.from_edge_lists(570, slices, name="cliques"), F(1, 2))
    _same(g, gamma=gamma, max_iterations=2, seed=1)
    _same(g, gamma=gamma, max_iterations=2, seed=1, initial=np.zeros(2280, np.int32))
    g.close()
