"""The workloads that the library's speed is judged on: solves of resident graphs (small to
large, every objective, weights, warm starts, general coupling), batched and served solves,
windowed long sequences, the graph build with the Bethe-Hessian operator, and the spectral
pathway.  Sizes follow the shapes of ``gen`` (the planted partition, the SBM rows, the weighted
and the heavy-tailed DC-SBM, the batch's shapes, the long sequences); inputs are drawn from a
seed with the DC-SBM law of ``gen.dcsbm``, on the GPU.
"""
import math
from fractions import Fraction

import numpy as np
import torch

from paper_2608_03695_amd import gen, mslm

LONG_WINDOW = gen.LONG_WINDOW   # snapshots per window, overlapping snapshots
SERVE_BUDGET = 64 << 30         # device bytes the request loop may hold


# ----------------------------------------------------------------------------- the cases

def _solve(n, t, degree, k, mu=0.3, alpha=2.5, churn=0.05, weights=1, gamma="1", omega="1",
           null=mslm.MSLM_NULL_MULTISLICE, slices=False, warm=False, coupling="ordinal",
           absent=0.0, static=False, **extra):
    return dict(kind="solve", n=n, t=t, degree=float(degree), k=k, mu=mu, alpha=alpha,
                churn=churn, weights=weights, gamma=gamma, omega=omega, null=null, slices=slices,
                warm=warm, coupling=coupling, absent=absent, static=static, **extra)


def listed():
    glob, cpm = mslm.MSLM_NULL_GLOBAL, mslm.MSLM_NULL_CPM
    return [
        dict(_solve(1000, 4, 7, 10), name="solve_planted_1k_x4", planted=True),
        dict(_solve(50_000, 5, 10, 10), name="solve_sbm_50k_x5"),
        dict(_solve(100_000, 16, 16, 100, weights=8), name="solve_weighted_100k_x16"),
        dict(_solve(100_000, 32, 10, 100, mu=0.4, alpha=2.1, churn=0.02, omega="1/2"),
             name="solve_heavy_100k_x32"),
        dict(_solve(50_000, 10, 10, 10, null=glob), name="solve_global_50k_x10"),
        dict(_solve(20_011, 7, 16, 40, null=cpm, gamma="1/1000"), name="solve_cpm_20k_x7"),
        dict(_solve(30_000, 12, 12, 60, slices=True, warm=True, coupling="categorical",
                    absent=0.2), name="solve_warm_categorical_30k_x12"),
        dict(kind="batch", first=0, graphs=8, gammas="1", omegas="1/10,1,10",
             name="batch_8_graphs_x3"),
        dict(kind="serve", first=64, requests=12, name="serve_12_requests"),
        dict(kind="windowed", n=327, t=400, edges=28, k=10, mu=0.3, alpha=2.5, churn=0.01,
             name="windowed_school_327_x400"),
        dict(kind="build", n=100_000, t=16, degree=16.0, k=100, mu=0.3, alpha=2.5, churn=0.05,
             weights=8, omega="1", r=3.7, name="build_apply_100k_x16"),
        dict(kind="spectral", n=50_000, t=8, degree=16.0, k=100, mu=0.3, alpha=2.5, churn=0.05,
             weights=8, omega="1", vectors=8, name="spectral_50k_x8"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve"] * 5 + ["batch", "serve", "windowed", "build", "spectral"])
    if kind == "batch":
        return dict(kind=kind, first=rng.randrange(500), graphs=rng.randint(2, 6),
                    gammas=rng.choice(["1", "1/2,2"]), omegas=rng.choice(["1", "1/10,10"]))
    if kind == "serve":
        return dict(kind=kind, first=rng.randrange(480), requests=rng.randint(2, 12))
    if kind == "windowed":
        n = _log_int(rng, 300, 12_500)
        return dict(kind=kind, n=n, t=_log_int(rng, 65, 400 if n < 2000 else 180),
                    edges=rng.randint(20, 60), k=rng.choice([10, 60]), mu=rng.choice([0.2, 0.3]),
                    alpha=rng.choice([2.1, 2.5]), churn=0.01)
    t = _log_int(rng, 2, 64)
    degree = round(rng.uniform(4, 24), 1)
    n = _log_int(rng, 300, min(100_000, 1_200_000 // t, int(12_000_000 / (t * degree))))
    base = dict(n=n, t=t, degree=degree, k=max(2, round(math.sqrt(n))),
                mu=round(rng.uniform(0.1, 0.5), 2), alpha=rng.choice([2.1, 2.5]),
                churn=rng.choice([0.02, 0.05, 0.1]), weights=rng.choice([1, 1, 8]),
                omega=rng.choice(["1/10", "1/2", "1", "10"]))
    if kind == "build":
        return dict(base, kind=kind, r=round(rng.uniform(1.0, 6.0), 2))
    if kind == "spectral":
        return dict(base, kind=kind, vectors=rng.choice([4, 8, 10]))
    null = rng.choice([mslm.MSLM_NULL_MULTISLICE] * 3 + [mslm.MSLM_NULL_GLOBAL, mslm.MSLM_NULL_CPM])
    case = _solve(**dict(base, null=null, gamma=rng.choice(["1/2", "1", "2"])))
    if null == mslm.MSLM_NULL_GLOBAL:
        case["weights"] = 1
    elif null == mslm.MSLM_NULL_CPM:
        case["n"], case["gamma"] = min(n, 150_000 // t), rng.choice(["1/1000", "1/100"])
    else:
        case["slices"] = rng.random() < 0.3
    case["warm"] = rng.random() < 0.3
    if t <= 12:
        case["coupling"] = rng.choice(["ordinal", "ordinal", "categorical"])
    case["absent"] = rng.choice([0.0, 0.0, 0.2])
    case["static"] = n * t <= 20_000 and rng.random() < 0.5
    return case


# ----------------------------------------------------------------------------- inputs

def _planted_labels(n, t, k, churn, rng):
    """Communities of every snapshot: Pareto sizes, floor(churn n) movers per transition."""
    labels = np.repeat(np.arange(k), gen._community_sizes(n, k, rng))[rng.permutation(n)]
    out = np.empty((t, n), np.int64)
    movers = int(math.floor(churn * n))
    for s in range(t):
        if s and movers:
            labels = labels.copy()
            who = rng.choice(n, size=movers, replace=False)
            labels[who] = labels[rng.integers(0, n, movers)]
        out[s] = labels
    return out


def _dcsbm(n, t, degree, k, mu, alpha, churn, weights, absent, seed):
    """The DC-SBM law of gen.dcsbm, all snapshots at once on the GPU: a pair's first end is
    drawn by propensity, its second end inside the first one's community with probability
    1 - mu, else outside it; self-pairs and repeats are dropped; a node is absent from a snapshot
    (all its edges dropped there) with probability `absent`."""
    rng = np.random.default_rng(seed)
    theta = gen._powerlaw_propensity(n, alpha, degree, rng)
    planted = _planted_labels(n, t, k, churn, rng)
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    rand = lambda m: torch.rand(m, generator=g, device=dev, dtype=torch.float64)   # noqa: E731
    weight = torch.from_numpy(np.maximum(1, np.rint(theta * 65536)).astype(np.int64)).to(dev)
    lab = torch.from_numpy(planted).to(dev)
    block = (lab + k * torch.arange(t, device=dev)[:, None]).reshape(-1)   # (snapshot, community)
    order = torch.argsort(block, stable=True)
    zero = torch.zeros(1, dtype=torch.int64, device=dev)
    cum = torch.cat([zero, torch.cumsum(weight.repeat(t)[order], 0)])
    end = torch.cumsum(torch.bincount(block, minlength=t * k), 0)
    before = cum[torch.cat([zero, end[:-1]])]
    total = cum[end] - before
    whole = torch.cumsum(weight, 0)
    pairs = int(round(n * degree / 2))
    m = pairs * t
    snap = torch.arange(t, device=dev).repeat_interleave(pairs)

    def anyone(count):
        at = (rand(count) * whole[-1].double()).long().clamp_(max=int(whole[-1]) - 1)
        return torch.searchsorted(whole, at, right=True)

    u = anyone(m)
    bu = block[snap * n + u]
    at = before[bu] + torch.minimum((rand(m) * total[bu].double()).long(), total[bu] - 1)
    x = order[torch.searchsorted(cum[1:], at, right=True)] % n
    away = rand(m) < mu
    far = anyone(m)
    for _ in range(6):
        far = torch.where(block[snap * n + far] == bu, anyone(m), far)
    x = torch.where(away, far, x)
    keep = u != x
    if absent > 0:
        gone = torch.rand((t, n), generator=g, device=dev) < absent
        keep &= ~(gone[snap, u] | gone[snap, x])
    u, x, snap = u[keep], x[keep], snap[keep]
    key = torch.unique((snap * n + torch.minimum(u, x)) * n + torch.maximum(u, x))
    key = key[torch.randperm(key.numel(), generator=g, device=dev)]   # edges in no order
    key = key[torch.argsort(key // (n * n), stable=True)]
    snap, u, x = key // (n * n), key // n % n, key % n
    flip = rand(key.numel()) < 0.5
    src, dst = torch.where(flip, x, u), torch.where(flip, u, x)
    w = None
    if weights > 1:
        w = torch.randint(1, weights + 1, (key.numel(),), generator=g, device=dev,
                          dtype=torch.int32).cpu().numpy()
    offsets = np.zeros(t + 1, np.int64)
    offsets[1:] = np.cumsum(torch.bincount(snap, minlength=t).cpu().numpy())
    return gen.TemporalGraph(n, t, offsets, src.int().cpu().numpy(), dst.int().cpu().numpy(), w,
                             planted.astype(np.int32))


def _case_graph(case, seed):
    if case.get("planted"):
        return gen.planted_partition(case["n"], case["t"], case["k"], 0.05, 0.002, 0.10, seed=seed)
    return _dcsbm(case["n"], case["t"], case["degree"], case["k"], case["mu"], case["alpha"],
                  case["churn"], case["weights"], case.get("absent", 0.0), seed)


def _batch_graphs(case, count, seed):
    """Graphs of the batched workload's shapes (gen.batch_graph_shape), from `first` on."""
    out = []
    for i in range(count):
        n, t, degree, mu = gen.batch_graph_shape((case["first"] + i) % 512)
        k = max(2, int(round(math.sqrt(n))))
        out.append(_dcsbm(n, t, degree, k, mu, 2.5, 0.05, 1, 0.0, seed * 1000 + i))
    return out


def _coupling(case):
    if case.get("coupling") != "categorical":
        return None
    return 1 - np.eye(case["t"], dtype=np.int32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        tg = _case_graph(case, seed)
        graph = mslm.Graph(tg, Fraction(case["omega"]), coupling=_coupling(case),
                           present_only=case["absent"] > 0)
        kw = dict(gamma=Fraction(case["gamma"]), max_levels=32, max_iterations=2, seed=0,
                  null_model=case["null"], no_alloc=case["static"])
        if case["slices"]:
            kw["gamma_slices"] = [gen.GAMMA_GRID[s % 3] for s in range(case["t"])]
        if case["warm"]:   # resume from the generating communities, each copy's label below T*N
            kw["initial"] = tg.planted.reshape(-1).astype(np.int32)
        return dict(kind=kind, graph=graph, kw=kw)
    if kind == "batch":
        graphs = [mslm.Graph(tg, 1) for tg in _batch_graphs(case, case["graphs"], seed)]
        solves = [(i, Fraction(a), Fraction(b), 32, 2, 0) for i in range(len(graphs))
                  for a in case["gammas"].split(",") for b in case["omegas"].split(",")]
        return dict(kind=kind, graphs=graphs, solves=solves)
    if kind == "serve":
        graphs = _batch_graphs(case, case["requests"], seed)
        pick = np.random.default_rng(seed)
        specs = [(gen.GAMMA_GRID[int(pick.integers(0, 3))], gen.OMEGA_GRID[int(pick.integers(0, 3))])
                 for _ in graphs]
        return dict(kind=kind, server=mslm.Server(SERVE_BUDGET, 4), graphs=graphs, specs=specs)
    if kind == "windowed":
        n = case["n"]
        return dict(kind=kind, graph=_dcsbm(n, case["t"], 2.0 * case["edges"] / n, case["k"],
                                            case["mu"], case["alpha"], case["churn"], 1, 0.0, seed))
    tg = _case_graph(case, seed)
    if kind == "build":
        x = np.random.default_rng(seed).standard_normal(tg.n_supra)
        return dict(kind=kind, tg=tg, omega=Fraction(case["omega"]), r=case["r"], x=x)
    return dict(kind=kind, graph=mslm.Graph(tg, Fraction(case["omega"])), k=case["vectors"])


# ----------------------------------------------------------------------------- one pass

_COUNTS = ("q", "n_communities", "levels_run", "iterations_run", "colours_level0", "sweeps", "moves",
           "refine_rounds", "merges", "splits")


def _solved(memb, res):
    return {"membership": memb, "q_components": res["q_components"],
            **{key: res[key] for key in _COUNTS}}


def _together(results):
    """Several solves' outputs, joined (memberships end to end, one row of counts each)."""
    outs = [_solved(memb, res) for memb, res in results]
    return {key: (np.concatenate([o[key] for o in outs]) if key in ("membership", "q_components")
                  else np.array([o[key] for o in outs])) for key in outs[0]}


def run(state):
    kind = state["kind"]
    if kind == "solve":
        return _solved(*state["graph"].leiden(**state["kw"]))
    if kind == "batch":
        return _together(mslm.batch_leiden(state["graphs"], state["solves"]))
    if kind == "serve":
        server = state["server"]
        tickets = [server.submit(tg, gamma, omega)
                   for tg, (gamma, omega) in zip(state["graphs"], state["specs"])]
        return _together([server.wait(t)[:2] for t in tickets])
    if kind == "windowed":
        memb, res = mslm.leiden_windowed(state["graph"], 1, *LONG_WINDOW, gamma=1,
                                         max_iterations=2, present_only=True)
        return {"membership": memb, "n_communities": res["n_communities"]}
    if kind == "build":
        graph = mslm.Graph(state["tg"], state["omega"])
        y = graph.bh_apply(state["x"], state["r"])
        info = graph.info()
        graph.close()
        return {"y": y, **info}
    values, _, labels, res = state["graph"].bethe_hessian(state["k"], embedding=False, seed=1)
    return {"eigenvalues": values, "labels": labels, "r": res["r"],
            "lanczos_steps": res["lanczos_steps"]}


# ----------------------------------------------------------------------------- bytes, exact values

def _sizes(case):
    """(supra-nodes, directed intra entries, directed coupling entries) expected of a graph."""
    n, t = case["n"], case["t"]
    degree = 2.0 * case["edges"] / n if case["kind"] == "windowed" else case["degree"]
    present = (1.0 - case.get("absent", 0.0)) ** 2
    pairs = t * (t - 1) if case.get("coupling") == "categorical" else 2 * (t - 1)
    return n * t, n * t * degree * present, n * pairs * present


def work(case):
    """The graph read once and the outputs written once; two operations per entry."""
    kind = case["kind"]
    if kind in ("batch", "serve"):
        count = case["graphs"] if kind == "batch" else case["requests"]
        per = len(case["gammas"].split(",")) * len(case["omegas"].split(",")) if kind == "batch" else 1
        units = entries = 0.0
        for i in range(count):
            n, t, degree, _ = gen.batch_graph_shape((case["first"] + i) % 512)
            units += n * t
            entries += n * t * degree + 2 * n * (t - 1)
        return {"bytes": (4 * entries + 8 * units) + per * 4 * units, "flops": per * 2 * entries}
    units, intra, inter = _sizes(case)
    entry = 8 if case.get("weights", 1) > 1 else 4
    graph = entry * (intra + inter) + 8 * units
    if kind == "build":   # edge lists in, the two vectors of the operator
        return {"bytes": (entry + 4) * intra / 2 + 16 * units, "flops": 2 * (intra + inter)}
    if kind == "spectral":
        return {"bytes": graph + 4 * units, "flops": 2 * (intra + inter) * (case["vectors"] + 152)}
    if kind == "windowed":
        graph = 8 * intra / 2
    return {"bytes": graph + 4 * units, "flops": 2 * (intra + inter)}


def exact(case, seed):
    """y = H(r) x of the operator in float64 from the edge lists; the other outputs are whole
    numbers, or have no value short of the library's own schedule."""
    if case["kind"] != "build":
        return None
    tg = _case_graph(case, seed)
    n, t = case["n"], case["t"]
    x = np.random.default_rng(seed).standard_normal(n * t)
    base = np.repeat(np.arange(t) * n, np.diff(tg.offsets))
    u, v = base + tg.src, base + tg.dst
    w = np.ones(u.size) if tg.weight is None else tg.weight.astype(np.float64)
    d = np.bincount(u, w, n * t) + np.bincount(v, w, n * t)
    ax = np.bincount(u, w * x[v], n * t) + np.bincount(v, w * x[u], n * t)
    omega = float(Fraction(case["omega"]))
    xs, ds, axs = x.reshape(t, n), d.reshape(t, n), ax.reshape(t, n)
    ds[1:] += omega
    ds[:-1] += omega
    axs[1:] += omega * xs[:-1]
    axs[:-1] += omega * xs[1:]
    r = case["r"]
    return {"y": (r * r - 1.0 + d) * x - r * ax, "n_supra": None, "nnz": None, "two_m": None}
