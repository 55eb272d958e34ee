"""GPU: the work counters of a counting solve are those of the schedule, not of colours decided
ahead in vain: with one sweep a level every unit of every level is decided once and its row scanned
once, whatever the width of the windows, in plain and in counted solves alike."""
from fractions import Fraction as F

import numpy as np
import pytest

import oracle
from paper_2608_03695_amd import gen

pytestmark = pytest.mark.gpu


def _hubs():
    """A node of 5200 neighbours, so that every kind of unit occurs at level 0."""
    base = gen.dcsbm(6000, 2, 6, 60, 0.2, 2.5, 0.05, seed=5)
    rng = np.random.default_rng(4)
    slices = []
    for s in range(2):
        u, x, _ = base.slice_edges(s)
        slices.append([(int(a), int(b)) for a, b in zip(u, x)] +
                      [(0, int(b)) for b in rng.choice(np.arange(1, 6000), 5200, replace=False)])
    return gen.from_edge_lists(6000, slices, name="hubs")


# two slices: their totals have a common multiple that a double holds, so no sweep is repeated
GRAPHS = [("planted", lambda: gen.planted_partition(600, 2, 8, 0.08, 0.004, 0.1, seed=3), F(10)),
          ("dcsbm", lambda: gen.dcsbm(20000, 2, 10, 40, 0.3, 2.3, 0.03, seed=10), F(1, 2)),
          ("hubs", _hubs, F(1))]


@pytest.mark.parametrize("name,make,omega", GRAPHS, ids=[g[0] for g in GRAPHS])
def test_single_sweeps_count_every_unit_once(name, make, omega):
    from paper_2608_03695_amd import mslm
    tg = make()
    oracle.trace_enable(True)
    om, _, _ = oracle.OracleGraph(tg, omega).leiden(1, max_levels=32, max_iterations=1,
                                                    max_sweeps=1, seed=0)
    levels = oracle.trace_levels(tg.n_supra)
    oracle.trace_enable(False)
    assert len(levels) >= 3
    g = mslm.Graph(tg, omega)
    for tu in (dict(), dict(lat_parts_max=1), dict(split_group_units=0, latency_units=64),
               dict(split_group_units=1 << 30, latency_units=65536), dict(graphs=1)):
        g.set_tuning(**{**g.tuning(), **tu})
        m, r = g.leiden(1, max_iterations=1, max_sweeps=1, count=True)
        assert np.array_equal(m, om), tu
        assert (r["lm0_units"], r["lm0_entries"]) == (levels[0]["n"], levels[0]["nnz"]), tu
        assert (r["lm_units"], r["lm_entries"]) == (sum(lv["n"] for lv in levels),
                                                    sum(lv["nnz"] for lv in levels)), tu
        assert 0 < r["lm0_candidates"] <= r["lm0_entries"], tu
        assert r["lm0_candidates"] <= r["lm_candidates"] <= r["lm_entries"], tu
    g.close()


def test_later_sweeps_count_at_most_every_unit_once():
    """Units at rest are not decided: several sweeps count no more than all units in each."""
    from paper_2608_03695_amd import mslm
    g = mslm.Graph(gen.dcsbm(20000, 2, 10, 40, 0.3, 2.3, 0.03, seed=10), F(1, 2))
    info = g.info()
    for parts in (1, 16):
        g.set_tuning(lat_parts_max=parts)
        _, r = g.leiden(1, max_levels=1, count=True)
        _, plain = g.leiden(1, max_levels=1)
        assert r["moves"] == plain["moves"] and plain["lm0_units"] == 0
        assert 2 * info["n_supra"] <= r["lm0_units"] <= r["sweeps"] * info["n_supra"]
        assert r["lm0_entries"] <= r["sweeps"] * info["nnz"]
    g.close()
