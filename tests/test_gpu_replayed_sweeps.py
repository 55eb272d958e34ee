"""GPU: sweeps replayed from a captured HIP graph (tuning graphs = 1) where the sweeps of one level
go back and forth between few moves and many (above and below a 32nd of the level's units, at which
records of units at rest are kept) and near-ties have sweeps taken again: memberships, Q components
and statistics must equal the oracle's.

The graphs are unions of matchings, each edge weight used in two snapshots: every node has much the
same degree everywhere, so gains tie often, and the snapshot totals have no common multiple below
2^53, so that the ties are near-ties of the double estimates.  At one level of the graph RISING the
moves go 73, 3, 2, 11, 20, 12, 8, 8, 25, ...: in a union its copies hold every sweep from the fifth
on to many moves, while the sweeps of the graph TIED are taken again and its units go on moving."""
from fractions import Fraction as F

import numpy as np
import pytest

import oracle
from paper_2608_03695_amd import gen

pytestmark = pytest.mark.gpu

WEIGHTS = [97, 101, 103, 107, 109, 113, 127, 131]
STAT_KEYS = ["sweeps", "moves", "sweep_cap_hits", "refine_rounds", "merges", "splits",
             "levels_run", "iterations_run", "n_communities"]


def _matching(rng, n, order, blocks, inside):
    """Pairs of nodes: mostly inside blocks of `order` with probability `inside`, else any."""
    if rng.random() < inside:
        perm = np.argsort(order // max(1, n // blocks) + rng.random(n) * rng.choice([0.5, 1.5, 3.0]))
    else:
        perm = rng.permutation(n)
    return [(int(perm[i]), int(perm[i + 1])) for i in range(0, n - 1, 2)]


def _simple(seed):
    """Pairs drawn twice in a snapshot count once."""
    rng = np.random.default_rng(seed)
    n, used, count, blocks = (int(rng.integers(*x)) for x in ((24, 90), (7, 9), (1, 4), (2, 8)))
    order, slices = rng.permutation(n), []
    for w in WEIGHTS[:used]:
        for _ in range(2):
            pairs = [p for _ in range(count) for p in _matching(rng, n, order, blocks, 0.6)]
            slices.append([(*p, w) for p in sorted({(min(p), max(p)) for p in pairs})])
    return gen.from_edge_lists(n, slices, weighted=True, name="simple")


def _repeated(seed):
    """Pairs drawn twice in a snapshot count twice: all degrees of a snapshot are equal."""
    rng = np.random.default_rng(seed)
    n = int(rng.choice([12, 16, 18, 20, 24, 30, 32, 36, 40, 48, 60, 64, 72]))
    used, count, blocks = (int(rng.integers(*x)) for x in ((7, 9), (1, 5), (2, 8)))
    order, inside, slices = rng.permutation(n), rng.choice([0.3, 0.6, 0.9]), []
    rng.random()
    for w in WEIGHTS[:used]:
        for _ in range(2):
            slices.append([(*p, w) for _ in range(count)
                           for p in _matching(rng, n, order, blocks, inside)])
    return gen.from_edge_lists(n, slices, weighted=True, name="repeated")


RISING = (_simple(3001989), F(1, 2), F(400), 4)
TIED = (_repeated(2806303), F(2), F(30), 1)
# levels whose moves rise again after few, near-ties among them: alone, three iterations each
ALONE = [(_simple(16877), F(1, 2), F(400), 0), (_simple(9408), F(1, 2), F(60), 4),
         (_simple(806945), F(1, 2), F(400), 3), (_repeated(3001234), F(1), F(10), 0)]
TUNINGS = [dict(graphs=1), dict(graphs=1, lat_parts_max=1), dict(graphs=1, latency_units=64),
           dict(graphs=0)]


def _check(got, want, case):
    om, oc, ost = want
    m, r = got
    assert np.array_equal(m, om), case
    assert np.array_equal(r["q_components"], oc), case
    for k in STAT_KEYS:
        assert r[k] == ost[k], (case, k)


def _oracle(tg, gamma, omega, seed, iterations):
    return oracle.OracleGraph(tg, omega).leiden(gamma, max_levels=32, max_iterations=iterations,
                                                seed=seed)


@pytest.mark.parametrize("copies", [20, 60])
def test_union_whose_moves_rise_again_matches_oracle(copies):
    from paper_2608_03695_amd import mslm
    want = [_oracle(*c, 1) for c in (RISING, TIED)]
    handles = [mslm.Graph(c[0], c[2]) for c in (RISING, TIED)]
    which = [0] * copies + [1]
    solves = [(i, (RISING, TIED)[i][1], (RISING, TIED)[i][2], 32, 1, (RISING, TIED)[i][3])
              for i in which]
    for tu in TUNINGS:
        handles[0].set_tuning(**tu)
        for i, got in zip(which, mslm.batch_leiden(handles, solves)):
            _check(got, want[i], (tu, i))
    for h in handles:
        h.close()


@pytest.mark.parametrize("case", ALONE, ids=["rising", "endless", "long", "dense"])
def test_solves_whose_moves_rise_again_match_oracle(case):
    from paper_2608_03695_amd import mslm
    tg, gamma, omega, seed = case
    want = _oracle(*case, 3)
    g = mslm.Graph(tg, omega)
    for tu in TUNINGS:
        g.set_tuning(**tu)
        _check(g.leiden(gamma, max_iterations=3, seed=seed), want, tu)
    g.close()
