"""The calls whose speed matters, over the sizes that users bring.

Every case goes through the public entry points as a program calls them:
whole layouts decomposed (graph or rectangles in hand), a resident batch
solved again, components given directly, requests served.  Layouts come from
the seeded generator, with the densities, distances, mask counts and budgets
of the repository's own workloads; only their sizes and seeds vary.
"""
from __future__ import annotations

import math

import numpy as np

import paper_2303_14335_amd as mp
import workload

# Rectangles per square micrometre and minimum coloring distance of the three
# kinds of layout: triple patterning (sparse), quadruple patterning with every
# rectangle longer than 120 nm split at its middle, and a packed window that
# is one giant component.
KINDS = {
    "k3": dict(k=3, dmin=80, split=0, budget=1_000_000),
    "k4": dict(k=4, dmin=120, split=120, budget=1_000_000),
    "giant": dict(k=3, dmin=100, split=0, budget=10_000_000),
}


def listed():
    return [
        # one small window (an interactive edit, a cell): latency of a call
        dict(name="decompose_300_k3", do="decompose", kind="k3", rects=300, density=33.3),
        # a block of a chip, triple patterning: many tiny components
        dict(name="decompose_200k_k3", do="decompose", kind="k3", rects=200_000, density=20.0),
        # the same block for quadruple patterning with stitches: components
        # of up to a few dozen nodes, some with long searches
        dict(name="decompose_200k_k4_stitch", do="decompose", kind="k4", rects=200_000, density=20.0),
        # a packed window: one component of 40k nodes
        dict(name="decompose_40k_giant", do="decompose", kind="giant", rects=39_983, density=277.0),
        # rectangles in, colors out: the graph built on the device first
        dict(name="layout_50k_k3", do="layout", kind="k3", rects=50_001, density=33.3),
        # the front-end alone, for a program with its own solver or for
        # planning: layout graph and its split into components
        dict(name="front_end_200k_k4", do="front_end", kind="k4", rects=200_000, density=20.0),
        # a batch kept on the device and solved again
        dict(name="batch_200k_k3", do="batch", kind="k3", rects=200_000, density=20.0),
        # every node colored at least cost: stitch-aware search, conflict
        # marking and the minimisation of conflicts and stitches
        dict(name="minimize_30k_k4", do="minimize", kind="k4", rects=30_001, density=20.0),
        # components of a caller's own split, nothing allocated on the way
        dict(name="components_small", do="noalloc", k=3, count=65, n_min=4, n_max=24, degree=3.6,
             budget=1_000_000, trace=False),
        # mid-sized components near the coloring threshold (most are colored
        # at once, about a third run to the budget), with the trace hash that
        # a regression check compares
        dict(name="components_mid", do="components", k=3, count=48, n_min=65, n_max=2048, degree=4.2,
             budget=100_000, trace=True),
        # large components whose search runs to its budget
        dict(name="components_big", do="components", k=3, count=3, n_min=4000, n_max=10_000, degree=4.3,
             budget=50_000, trace=False),
        # a burst of layouts at the server, submitted together
        dict(name="serve_48", do="serve", kind="k3", count=48, n_min=100, n_max=50_000, density=33.3),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    do = rng.choice(["decompose", "decompose", "layout", "front_end", "batch", "minimize", "noalloc",
                     "components", "components", "serve"])
    if do == "noalloc":
        return dict(do=do, k=rng.choice([3, 4]), count=log_int(1, 500), n_min=4, n_max=rng.randint(8, 64),
                    degree=round(rng.uniform(3.2, 4.0), 2), budget=10_000, trace=rng.random() < 0.5)
    if do == "components":
        if rng.random() < 0.5:
            return dict(do=do, k=3, count=log_int(1, 48), n_min=65, n_max=log_int(130, 2048),
                        degree=round(rng.uniform(3.8, 4.5), 2), budget=log_int(1000, 100_000),
                        trace=rng.random() < 0.5)
        return dict(do=do, k=3, count=rng.randint(1, 3), n_min=2049, n_max=log_int(3000, 10_000),
                    degree=round(rng.uniform(3.9, 4.5), 2), budget=log_int(1000, 50_000),
                    trace=rng.random() < 0.5)
    if do == "serve":
        return dict(do=do, kind="k3", count=log_int(2, 48), n_min=100, n_max=log_int(1000, 50_000),
                    density=33.3)
    if do == "decompose" and rng.random() < 0.3:
        return dict(do=do, kind="giant", rects=log_int(2000, 39_900), density=277.0)
    if do == "minimize":
        return dict(do=do, kind=rng.choice(["k3", "k4"]), rects=log_int(300, 30_000), density=20.0)
    kind = "k3" if do == "batch" else rng.choice(["k3", "k4"])
    density = round(rng.uniform(18.0, 34.0) if kind == "k3" else rng.uniform(15.0, 20.0), 1)
    return dict(do=do, kind=kind, rects=log_int(300, 190_000), density=density)


# ---- inputs -------------------------------------------------------------

def _mix(seed, i=0):
    """A layout seed of its own for each (seed, request)."""
    return workload.splitmix64(seed * 1_000_003 + i, 1)[0]


def _layout(rects, density, seed):
    side = int(round(1000.0 * math.sqrt(rects / density)))
    return workload.generate(rects, max(side, 300), seed)[0]


def _component(n, degree, rng):
    """A connected random graph: a path and random pairs beside it."""
    m = max(n - 1, int(n * degree / 2))
    path = np.stack([np.arange(n - 1), np.arange(1, n)], 1)
    seen = set((path[:, 0] * n + path[:, 1]).tolist())
    most = n * (n - 1) // 2
    codes = list(seen)
    while len(codes) < min(m, most):
        ab = np.sort(rng.integers(0, n, (2 * (m - len(codes)) + 8, 2)), axis=1)
        for c in (ab[:, 0] * n + ab[:, 1])[ab[:, 0] < ab[:, 1]].tolist():
            if c not in seen and len(codes) < min(m, most):
                seen.add(c)
                codes.append(c)
    codes = np.sort(np.array(codes, np.int64))
    return n, np.stack([codes // n, codes % n], 1).astype(np.int32)


def _sizes(case):
    """`count` sizes from n_min to n_max, even over their logarithm, odd and
    even ones in no order."""
    at = (np.arange(case["count"]) * 0.6180339887498949 + 0.5) % 1.0
    return np.floor(np.exp(math.log(case["n_min"]) + at * math.log((case["n_max"] + 1) / case["n_min"]))).astype(int)


_contexts: dict = {}
_servers: list = []


def _context(of="calls"):
    """One context for a program's calls, one that its server owns."""
    if of not in _contexts:
        _contexts[of] = mp.Context(0)
    return _contexts[of]


def _server():
    if not _servers:
        _servers.append(mp.Server(_context("server")))
    return _servers[0]


def prepare(case, seed):
    do = case["do"]
    if do in ("noalloc", "components"):
        rng = np.random.default_rng(_mix(seed))
        return dict(case=case, ctx=_context(),
                    comps=[_component(int(n), case["degree"], rng) for n in _sizes(case)])
    p = KINDS[case["kind"]]
    if do == "serve":
        return dict(case=case, p=p, server=_server(),
                    layouts=[_layout(int(n), case["density"], _mix(seed, 1 + i))
                             for i, n in enumerate(_sizes(case))])
    rects = _layout(case["rects"], case["density"], _mix(seed))
    state = dict(case=case, p=p, ctx=_context(), rects=rects)
    if do in ("decompose", "minimize", "batch"):
        state["graph"] = mp.mpld_build_graph(rects, p["dmin"], p["split"])
    if do == "batch":
        state["batch"] = mp.Batch(state["ctx"], state["graph"], p["k"], p["budget"])
    return state


# ---- one pass -----------------------------------------------------------
# How many nodes, pairs and components a layout has differs from seed to
# seed: those outputs are returned whole at the front of an array whose
# length the case alone fixes, -1 behind them.

def _fixed(a, size):
    out = np.empty((size,) + a.shape[1:], a.dtype)
    out[: len(a)] = a
    out[len(a):] = -1
    return out


def _records(recs, size=None):
    recs = recs if size is None else _fixed(recs.view(np.int32).reshape(len(recs), 12), size).view(recs.dtype)[:, 0]
    out = {f: recs[f] for f in recs.dtype.names if f != "trace_hash"}
    out["trace_hash"] = recs["trace_hash"].view(np.int64)
    return out


def _result(case, r):
    n = case["rects"] * (2 if KINDS[case["kind"]]["split"] else 1)
    return dict(colors=_fixed(r.colors, n), component_of=_fixed(r.component_of, n), stitches=r.stitches,
                conflicts=r.conflicts, uncolored=r.uncolored, components=len(r.components),
                records=_records(r.components, 64 + n // 16))


def run(state):
    case, do = state["case"], state["case"]["do"]
    if do in ("noalloc", "components"):
        solve = mp.mpld_solve_components_noalloc if do == "noalloc" else mp.mpld_solve_components
        recs, cols = solve(state["ctx"], state["comps"], case["k"], case["budget"],
                           mp.MPLD_TRACE_HASH if case["trace"] else 0)
        return dict(records=_records(recs), colors=np.concatenate(cols))
    p = state["p"]
    if do == "serve":
        tickets = [state["server"].submit_layout(r, p["dmin"], p["split"], p["k"], p["budget"])
                   for r in state["layouts"]]
        done = [state["server"].wait(t) for t in tickets]
        n = sum(len(r) for r in state["layouts"])
        return dict(colors=np.concatenate([r.colors for r in done]),
                    component_of=np.concatenate([r.component_of for r in done]),
                    records=_records(np.concatenate([r.components for r in done]), 64 + n // 16),
                    totals=np.array([[r.stitches, r.conflicts, r.uncolored, len(r.components)] for r in done]))
    ctx = state["ctx"]
    if do == "decompose":
        return _result(case, mp.mpld_decompose(ctx, state["graph"], p["k"], p["budget"]))
    if do == "minimize":
        flags = mp.MPLD_SIMPLIFY | mp.MPLD_STITCH_ORDER | mp.MPLD_MARK_CONFLICTS | mp.MPLD_MINIMIZE
        return _result(case, mp.mpld_decompose(ctx, state["graph"], p["k"], p["budget"], flags))
    if do == "layout":
        g = mp.mpld_build_graph_device(ctx, state["rects"], p["dmin"], p["split"])
        return _result(case, mp.mpld_decompose(ctx, g, p["k"], p["budget"]))
    if do == "front_end":
        g = mp.mpld_build_graph_device(ctx, state["rects"], p["dmin"], p["split"])
        removal, comp_of, comps = mp.mpld_split_graph_device(ctx, g, p["k"])
        n = case["rects"] * (2 if p["split"] else 1)
        pairs = int(1.5 * _graph_size(case["rects"], case["density"], p)[1]) + 64
        sizes = np.array([len(c) for c in comps], np.int32)
        order = np.concatenate(comps) if comps else np.zeros(0, np.int32)
        return dict(conflict_pairs=_fixed(g.ce, pairs), stitch_pairs=_fixed(g.se, case["rects"]),
                    removal=_fixed(removal, n), component_of=_fixed(comp_of, n),
                    sizes=_fixed(sizes, 64 + n // 16), order=_fixed(order, n))
    state["batch"].solve()
    return _result(case, state["batch"].result())


# ---- what a pass cannot do without --------------------------------------

def _graph_size(rects, density, p):
    """Nodes and conflict pairs to be expected of such a layout: a pair
    conflicts when one lies in the other's surroundings of width dmin
    (mean length 120, 81 when split, width 20)."""
    nodes = rects * (1.48 if p["split"] else 1.0)
    length = 81.0 if p["split"] else 120.0
    area = (4.0 * (length + 20.0) * p["dmin"] + math.pi * p["dmin"] ** 2) * 1e-6
    return nodes, nodes * nodes * area / (2.0 * rects / density)


def work(case):
    """Inputs read once and outputs written once; the search itself counts
    no floating-point operations."""
    do = case["do"]
    span = max(1e-9, math.log(case["n_max"] / case["n_min"])) if "n_max" in case else 1.0
    if do in ("noalloc", "components"):
        n = case["count"] * (case["n_max"] - case["n_min"]) / span
        return dict(bytes=n * (0.5 * case["degree"] * 8 + 1) + 48 * case["count"], flops=0)
    p = KINDS[case["kind"]]
    if do == "serve":
        rects = case["count"] * (case["n_max"] - case["n_min"]) / span
    else:
        rects = case["rects"]
    nodes, pairs = _graph_size(rects, case["density"], p)
    result = nodes * (1 + 4)
    stitch_pairs = 8 * (nodes - rects)
    if do == "front_end":
        return dict(bytes=16 * rects + 8 * pairs + stitch_pairs + nodes * 3 * 4, flops=0)
    if do in ("layout", "serve"):
        return dict(bytes=16 * rects + result, flops=0)
    if do == "batch":   # the packed components stay on the device
        return dict(bytes=result, flops=0)
    return dict(bytes=8 * pairs + stitch_pairs + result, flops=0)


def exact(case, seed):
    """Every output is a whole number, equal or wrong."""
    return None
