"""GPU: sweeps decide windows of several colours at once; memberships, Q components and the
schedule's statistics must equal the oracle's where a window can go wrong: more colours than a
wave has lanes, hub units (above the block table's 4096 entries) between ordinary ones, windows
as narrow and as wide as the tuning allows, one kernel for both unit classes or one each, tables
of every size, sweeps that skip units at rest, and unions of solves that stop at different
sweeps."""
from fractions import Fraction as F

import numpy as np
import pytest

import oracle
from paper_2608_03695_amd import gen

pytestmark = pytest.mark.gpu

STAT_KEYS = ["sweeps", "moves", "sweep_cap_hits", "refine_rounds", "merges", "splits",
             "levels_run", "iterations_run", "n_communities"]


def _dense():
    """More than 64 colours at level 0 and above (each snapshot holds cliques of 70 nodes)."""
    rng = np.random.default_rng(3)
    slices = []
    for _ in range(24):
        perm = rng.permutation(420)
        edges = [(int(perm[c * 70 + i]), int(perm[c * 70 + j])) for c in range(6)
                 for i in range(70) for j in range(i)]
        edges += [(int(a), int(b)) for a, b in rng.integers(0, 420, (2000, 2)) if a != b]
        slices.append(edges)
    return gen.from_edge_lists(420, slices, name="cliques")


def _hubs(degrees=(5200, 5200)):
    """Nodes of many neighbours in a graph of small communities."""
    base = gen.dcsbm(6000, 2, 6, 60, 0.2, 2.5, 0.05, seed=5)
    rng = np.random.default_rng(4)
    slices = []
    for s in range(2):
        u, x, _ = base.slice_edges(s)
        edges = [(int(a), int(b)) for a, b in zip(u, x)]
        for hub, d in enumerate(degrees):
            edges += [(hub, int(b)) for b in rng.choice(np.arange(len(degrees), 6000), d,
                                                             replace=False)]
        slices.append(edges)
    return gen.from_edge_lists(6000, slices, name="hubs")


GRAPHS = [("dense", _dense, F(1), F(1, 2)), ("hubs", _hubs, F(2), F(1)),
          # rows at the edges of the 2048-, 4096- and 8192-slot tables (a node's degree is about
          # its base degree above these)
          ("rows_2k", lambda: _hubs((1015, 1020, 1500, 1900)), F(2), F(1, 8)),
          ("rows_4k", lambda: _hubs((1015, 2030, 2045, 3900)), F(1, 2), F(1, 4))]
TUNINGS = [dict(), dict(lat_parts_max=1), dict(latency_units=64, split_group_units=0),
           dict(latency_units=65536, split_group_units=1 << 30, lat_parts_max=2)]


@pytest.mark.parametrize("name,make,gamma,omega", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_windows_match_oracle(name, make, gamma, omega):
    from paper_2608_03695_amd import mslm
    tg = make()
    om, oc, ost = oracle.OracleGraph(tg, omega).leiden(gamma, max_levels=32, max_iterations=2,
                                                       seed=0)
    g = mslm.Graph(tg, omega)
    default = g.tuning()
    for tu in TUNINGS:
        g.set_tuning(**default)
        g.set_tuning(**tu)
        m, r = g.leiden(gamma)
        assert np.array_equal(m, om), tu
        assert np.array_equal(r["q_components"], oc), tu
        for k in STAT_KEYS:
            assert r[k] == ost[k], (tu, k)
    g.set_tuning(**default)
    solves = [(0, gamma, omega, 32, 2, 0), (0, F(1, 2), F(10), 32, 1, 1), (0, gamma, omega, 2, 2, 0)]
    for sv, (m, r) in zip(solves, mslm.batch_leiden([g], solves)):
        pm, pr = g.leiden(sv[1], sv[2], max_levels=sv[3], max_iterations=sv[4], seed=sv[5])
        assert np.array_equal(m, pm), sv
        assert np.array_equal(r["q_components"], pr["q_components"]), sv
        for k in STAT_KEYS:
            assert r[k] == pr[k], (sv, k)
    g.close()


@pytest.mark.parametrize("cliques,size,slices", [(40, 24, 20), (1, 300, 30)],
                         ids=["chains", "beyond_the_planes"])
def test_colouring_matches_oracle(cliques, size, slices):
    """Colourings of more units than a wave, a block or the chip holds at once: many cliques (long
    chains of priorities side by side) and one of 300 nodes per snapshot, whose colours lie beyond
    the 64 that level 0 keeps in a bitmap and the 256 of an aggregated level; both above and, by
    the second solve's coupling-only graph, below the size at which chains are followed."""
    from paper_2608_03695_amd import mslm
    n = cliques * size
    edges = [(c * size + i, c * size + j) for c in range(cliques) for i in range(size)
             for j in range(i)]
    for name, per in (("all", [edges] * slices), ("few", [edges] * 2 + [[]] * 2)):
        tg = gen.from_edge_lists(n, per, name=name)
        om, oc, ost = oracle.OracleGraph(tg, 1).leiden(1, max_levels=32, max_iterations=1, seed=3)
        g = mslm.Graph(tg, 1)
        m, r = g.leiden(1, max_iterations=1, seed=3)
        g.close()
        assert np.array_equal(m, om), name
        assert np.array_equal(r["q_components"], oc), name
        assert r["colours_level0"] == ost["colours_first"], name
        for k in STAT_KEYS:
            assert r[k] == ost[k], (name, k)


@pytest.mark.parametrize("weight", [1, 1 << 10, 1 << 14, 1 << 18])
def test_common_denominators_match_oracle(weight):
    """Graphs full of exact ties (rings of equal cliques), with edge weights that take the values
    of targets, scaled by the slices' common denominator, from far below 2^53 (where doubles are
    exact) to beyond it, and slice totals with small and with large common multiples."""
    from paper_2608_03695_amd import mslm
    for extra in ((0, 0, 0), (0, 1, 5), (2, 3, 7)):
        slices = []
        for s in range(3):
            edges = [(c * 8 + i, c * 8 + j, weight) for c in range(15) for i in range(8)
                     for j in range(i)]
            edges += [(c * 8, (c * 8 + 9) % 120, weight) for c in range(15)]
            edges += [(c * 8 + 3, (c * 8 + 23) % 120, weight) for c in range(extra[s])]
            slices.append(edges)
        tg = gen.from_edge_lists(120, slices, weighted=True, name="ring")
        for omega, kw in ((F(1), {}), (F(1, 2), dict(gamma=F(1, 20), null_model=2))):
            om, oc, ost = oracle.OracleGraph(tg, omega).leiden(max_levels=32, max_iterations=2,
                                                               seed=1, **kw)
            g = mslm.Graph(tg, omega)
            m, r = g.leiden(max_iterations=2, seed=1, **kw)
            g.close()
            assert np.array_equal(m, om), (extra, omega)
            assert np.array_equal(r["q_components"], oc), (extra, omega)
            for k in STAT_KEYS:
                assert r[k] == ost[k], (extra, omega, k)


@pytest.mark.parametrize("n", [1, 2, 1023, 1024, 1025, 8191, 8192, 8193, 16383, 16384, 16385])
def test_sort_and_scan_sizes_match_oracle(n):
    """Levels of as many units, and entries, as one block sorts or scans, one fewer and one more."""
    from paper_2608_03695_amd import mslm
    rng = np.random.default_rng(n)
    ring = [(i, (i + 1) % n) for i in range(n)] if n > 2 else []
    far = rng.integers(0, n, (n // 2, 2))
    more = sorted({(min(a, b), max(a, b)) for a, b in far.tolist() if abs(a - b) > 2
                   and abs(a - b) < n - 2})
    tg = gen.from_edge_lists(n, [ring + more] if n > 2 else [[(0, 1)] * (n - 1)], name="ring")
    om, oc, ost = oracle.OracleGraph(tg, 1).leiden(1, max_levels=32, max_iterations=2, seed=2)
    g = mslm.Graph(tg, 1)
    m, r = g.leiden(1, seed=2)
    g.close()
    assert np.array_equal(m, om)
    assert np.array_equal(r["q_components"], oc)
    for k in STAT_KEYS:
        assert r[k] == ost[k], k


@pytest.mark.parametrize("gamma", [F(1, 4), F(200)], ids=["few", "many"])
def test_final_labels_match_oracle(gamma):
    """Final memberships of a handful of labels and of more than a block's label table holds, and
    communities that come apart into many trees of short and long rows."""
    from paper_2608_03695_amd import mslm
    tg = _hubs((1500, 5200))
    om, oc, ost = oracle.OracleGraph(tg, 1).leiden(gamma, max_levels=32, max_iterations=2, seed=4)
    g = mslm.Graph(tg, 1)
    m, r = g.leiden(gamma, seed=4)
    g.close()
    assert (r["n_communities"] > 1024) == (gamma == 200)
    assert np.array_equal(m, om)
    assert np.array_equal(r["q_components"], oc)
    for k in STAT_KEYS:
        assert r[k] == ost[k], k
