"""Components searched in pieces by many wavefronts (heavy-component solves of
the LDS and big tiers, and of register-tier components cut by their budget)
against the oracle: budgets on both sides of where pieces begin and end, piece
sizes from a few nodes (every piece cut again, and more pieces than there is
room for) to more than the search, every k, traced and not.  All outputs are
whole numbers: equal or wrong.
"""
import numpy as np
import pytest

import oracle
from algx_literal import random_graph

pytestmark = pytest.mark.gpu

TRACE, SIMPLIFY = 2, 0


def say(*a):
    print("[case]", *a, flush=True)


def component(n, degree, rng):
    e = {(i, i + 1) for i in range(n - 1)}
    want = min(max(int(n * degree / 2), n - 1), n * (n - 1) // 2)
    while len(e) < want:
        a, b = sorted(rng.integers(0, n, 2).tolist())
        if a != b:
            e.add((a, b))
    return n, np.array(sorted(e), np.int32)


def union(comps):
    at, ce = 0, []
    for n, e in comps:
        ce.append(e + at)
        at += n
    return at, np.concatenate(ce).astype(np.int32)


DEGREE = {2: 2.1, 3: 4.4, 4: 8.0, 5: 11.5, 6: 15.0, 7: 19.0, 8: 23.0}


@pytest.mark.parametrize("k", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("cap", [16, 48, 256, 5000])
def test_pieces_against_oracle(ctx, k, cap):
    import paper_2303_14335_amd as mp
    rng = np.random.default_rng(97 * k + cap)
    sizes = [40, 64, 65, 96, 97, 130, 257, 600] + ([2049, 2100] if k < 5 else [])
    n, ce = union([component(s, DEGREE[k] + 0.1 * (i % 4), rng) for i, s in enumerate(sizes)])
    se = np.zeros((0, 2), np.int32)
    for budget, trace in ((1, 1), (2, 0), (cap, 1), (cap + 1, 0), (3 * cap + 7, 1), (2500, 0), (6000, 1)):
        say("pieces", k, cap, budget, trace)
        ref = oracle.decompose(oracle.Graph(n, ce, se), k, budget, False)
        b = mp.Batch(ctx, mp.Graph(n, ce, se), k, budget, SIMPLIFY | (TRACE if trace else 0))
        b.set_tune(heavy_round_cap=cap, heavy_first_cap=64)
        for _ in range(2):
            b.solve(split=True)
            got = b.result()
            for f in ("status", "nodes", "depth_at_stop") + (("trace_hash",) if trace else ()):
                assert np.array_equal(got.components[f], ref.comps[f]), f
            assert np.array_equal(got.colors, ref.colors)
        b.close()


@pytest.mark.parametrize("tier", [0, 16, 32])
def test_every_budget(ctx, tier):
    """Each budget from 1 on, on a component that backtracks at once."""
    import paper_2303_14335_amd as mp
    rng = np.random.default_rng(5)
    comps = [component(s, 4.9, rng) for s in (24, 70, 110)]
    n, ce = union(comps)
    g = mp.Graph(n, ce, np.zeros((0, 2), np.int32))
    say("every budget, tier flag", tier)
    for budget in list(range(1, 160, 3)) + [511, 512, 513, 1777]:
        # the batch numbers each component from its smallest id, as the oracle's flow does
        ref = oracle.decompose(oracle.Graph(n, ce, np.zeros((0, 2), np.int32)), 3, budget, False)
        b = mp.Batch(ctx, g, 3, budget, TRACE | tier)
        b.set_tune(heavy_round_cap=16, heavy_first_cap=64)
        b.solve(split=True)
        got = b.result()
        b.close()
        for f in ("status", "nodes", "trace_hash", "depth_at_stop"):
            assert np.array_equal(got.components[f], ref.comps[f]), (budget, f)
        assert np.array_equal(got.colors, ref.colors)


@pytest.mark.parametrize("mib", [0, 2, 24, 200])
def test_little_memory(ctx, monkeypatch, mib):
    """The engine's workspace only as far as there is memory: the same answers
    with less of it or none, and all of it given back."""
    import torch

    import paper_2303_14335_amd as mp
    rng = np.random.default_rng(31)
    comps = [component(s, 4.4, rng) for s in (40, 64, 64, 300, 700, 2000, 3000)]
    say("little memory", mib)
    n, ce = union(comps)
    ref = oracle.decompose(oracle.Graph(n, ce, np.zeros((0, 2), np.int32)), 3, 20000, False)
    g = mp.Graph(n, ce, np.zeros((0, 2), np.int32))
    live = sum(t.numel() for t in ctx._alloc.live.values())
    empty, refused = torch.empty, []

    def limited(size, *args, **kw):
        # (the heavy-component engine's own areas, of at most 64 MiB, are not meant)
        if sum(t.numel() for t in ctx._alloc.live.values()) + size > live + (mib + 130 << 20):
            refused.append(size)
            raise torch.OutOfMemoryError("limited")
        return empty(size, *args, **kw)

    monkeypatch.setattr(torch, "empty", limited)
    got = mp.mpld_decompose(ctx, g, 3, 20000, TRACE)
    monkeypatch.undo()
    for f in ("status", "nodes", "trace_hash", "depth_at_stop"):
        assert np.array_equal(got.components[f], ref.comps[f]), f
    assert np.array_equal(got.colors, ref.colors)
    assert bool(refused) == (mib < 200)
    assert sum(t.numel() for t in ctx._alloc.live.values()) == live


def test_small_budgets(ctx):
    """On both sides of the budget from which components are searched in
    pieces (the largest one's nodes and ten shares)."""
    import paper_2303_14335_amd as mp
    rng = np.random.default_rng(12)
    n, ce = union([component(s, 4.5, rng) for s in (70, 300, 411)])
    g = mp.Graph(n, ce, np.zeros((0, 2), np.int32))
    for budget, pieces in ((411 + 2559, False), (411 + 2560, True)):
        say("small budgets", budget)
        ref = oracle.decompose(oracle.Graph(n, ce, np.zeros((0, 2), np.int32)), 3, budget, False)
        b = mp.Batch(ctx, g, 3, budget, TRACE)
        b.solve(split=True)
        got = b.result()
        for f in ("status", "nodes", "trace_hash", "depth_at_stop"):
            assert np.array_equal(got.components[f], ref.comps[f]), (budget, f)
        assert np.array_equal(got.colors, ref.colors)
        assert (b.info()["split_rounds"] > 0) == pieces
        b.close()
