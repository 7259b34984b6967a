"""Whole-layout decomposition of graphs large enough that the device
validates, splits, packs and recovers them, against the oracle: clusters on
both sides of every tier border, stitch pairs inside and across components,
each option, the batch calls on such a graph, and the graphs that the host
takes back (a fault, a hub, a recovery that is one long chain).  All outputs
are whole numbers: equal or wrong.
"""
import ctypes

import numpy as np
import pytest

import oracle
import workload
from algx_literal import random_graph

pytestmark = pytest.mark.gpu

SIMPLIFY, TRACE, FORCE_LDS, FORCE_GLOBAL = 1, 2, 16, 32
MARK, STITCH, MINIMIZE = 1 << 10, 1 << 11, 1 << 13


def say(*a):
    print("[case]", *a, flush=True)


def clustered(n, sizes, degree, stitch, seed):
    """n nodes with shuffled ids: a connected random graph on each cluster, a
    sparse forest-like rest tied to clusters and to itself, stitch pairs."""
    rng = np.random.default_rng(seed)
    ids = rng.permutation(n)
    pairs, at = set(), 0
    for s in sizes:
        e = {(i, i + 1) for i in range(s - 1)}
        want = min(max(int(s * degree / 2), s - 1), s * (s - 1) // 2)
        while len(e) < want:
            a, b = sorted(rng.integers(0, s, 2).tolist())
            if a != b:
                e.add((a, b))
        pairs |= {(at + a, at + b) for a, b in e}
        at += s
    for v in range(at, n):   # a few of the rest hang on anything before them
        if v and rng.random() < 0.7:
            pairs.add((int(rng.integers(0, v)), v))
    ce = np.array([(ids[a], ids[b]) for a, b in sorted(pairs)], np.int32).reshape(-1, 2)
    flip = rng.random(len(ce)) < 0.5
    ce[flip] = ce[flip][:, ::-1]
    ce = ce[rng.permutation(len(ce))]
    se = []
    if stitch:
        have = {tuple(sorted(p)) for p in ce.tolist()}
        perm = rng.permutation(n)[: n // 4 * 2].reshape(-1, 2)
        near = np.stack([ids[np.arange(0, at - 1, 2)], ids[np.arange(1, at, 2)]], 1)
        used = set()
        for a, b in np.concatenate([near, perm]).tolist():
            if a not in used and b not in used and tuple(sorted((a, b))) not in have:
                used |= {a, b}
                se.append((a, b))
    return n, ce, np.array(se, np.int32).reshape(-1, 2)


def compare(got, ref):
    assert np.array_equal(got.component_of, ref.comp_of)
    assert len(got.components) == len(ref.comps)
    for f in got.components.dtype.names:
        assert np.array_equal(got.components[f], ref.comps[f]), f
    assert np.array_equal(got.colors, ref.colors)
    assert (got.stitches, got.conflicts, got.uncolored) == (ref.stitches, ref.conflicts, ref.uncolored)


SMALL = [5, 6, 7, 30, 31, 63, 64, 64, 12, 9, 8] * 3
MIXED = SMALL + [65, 100, 700, 2047, 2048, 2049]


@pytest.mark.parametrize("k", [2, 3, 4, 6])
@pytest.mark.parametrize("n,sizes,flags", [
    (10000, SMALL, SIMPLIFY | TRACE), (10001, SMALL, TRACE), (9001, SMALL, SIMPLIFY | TRACE | STITCH),
    (20000, MIXED, SIMPLIFY | TRACE), (20001, MIXED, SIMPLIFY | TRACE | STITCH | MARK),
    (9002, SMALL, SIMPLIFY | TRACE | STITCH | MINIMIZE), (9003, SMALL, SIMPLIFY | TRACE | FORCE_LDS),
    (20000, [17] * 5 + [40] * 4, SIMPLIFY | TRACE),
    (6000, [600, 513, 900], SIMPLIFY | TRACE), (6000, [600, 513, 900, 700, 512], SIMPLIFY | TRACE),
    (9000, [4500, 800, 100], SIMPLIFY | TRACE | STITCH), (9010, [4200] + [600] * 4 + [80] * 5, TRACE)])
def test_clusters(ctx, k, n, sizes, flags):
    import paper_2303_14335_amd as mp
    degree = min(1.25 * k + 0.9, 2.3 * k - 2.0)
    say("clusters", k, n, len(sizes), flags)
    n, ce, se = clustered(n, sizes, degree, True, 7 * n + k)
    ref = oracle.decompose(oracle.Graph(n, ce, se), k, 300, bool(flags & SIMPLIFY), bool(flags & MARK),
                           bool(flags & STITCH), bool(flags & MINIMIZE), 60)
    got = mp.mpld_decompose(ctx, mp.Graph(n, ce, se), k, 300, flags, 60)
    compare(got, ref)
    b = mp.Batch(ctx, mp.Graph(n, ce, se), k, 300, flags, 60)
    for how in ({}, {"split": True}, {"roundtrip": True}):
        b.solve(**how)
        compare(b.result(), ref)
    if not flags & FORCE_LDS:   # laid out again with another schedule
        b.set_tune(order=1, waves_per_block=2, big_one_wave=0)
        b.solve(roundtrip=True)
        compare(b.result(), ref)
    b.close()


def test_no_pairs_and_no_core(ctx):
    import paper_2303_14335_amd as mp
    say("no pairs; a forest")
    none = np.zeros((0, 2), np.int32)
    n, ce, se = clustered(9500, [], 0, True, 3)
    for args in ((11000, none, none), (11001, none, np.array([[6499, 0]], np.int32)), (n, ce, se)):
        for flags in (SIMPLIFY | TRACE, TRACE):
            ref = oracle.decompose(oracle.Graph(*args), 3, 1000, bool(flags & SIMPLIFY))
            compare(mp.mpld_decompose(ctx, mp.Graph(*args), 3, 1000, flags), ref)


@pytest.mark.parametrize("order", ["up", "down", "zigzag"])
def test_long_chain(ctx, order):
    """Every node of a path waits for its neighbour: past the device's wait
    the host recovers it."""
    import paper_2303_14335_amd as mp
    n = 9001
    ids = {"up": np.arange(n), "down": np.arange(n)[::-1],
           "zigzag": np.argsort(np.concatenate([np.arange(0, n, 2), np.arange(1, n, 2)]))}[order]
    ce = np.stack([ids[:-1], ids[1:]], 1).astype(np.int32)
    se = np.stack([ids[0:n - 3:4], ids[2:n - 1:4]], 1).astype(np.int32)
    say("path", order)
    ref = oracle.decompose(oracle.Graph(n, ce, se), 3, 1000)
    b = mp.Batch(ctx, mp.Graph(n, ce, se), 3, 1000, SIMPLIFY | TRACE)
    for _ in range(2):
        b.solve()
        compare(b.result(), ref)
    b.close()


def test_hub(ctx):
    """Nodes of more neighbours than the device ranks: the host's graph."""
    import paper_2303_14335_amd as mp
    say("hubs of 2048, 2049 and 4000 neighbours")
    for d in (2048, 2049, 4000):
        hub = np.stack([np.zeros(d), np.arange(1, d + 1)], 1)
        ring = np.stack([np.arange(1, 400), np.arange(2, 401)], 1)
        ce = np.concatenate([hub, ring]).astype(np.int32)
        args = (11000, ce, np.array([[0, 6499]], np.int32))
        ref = oracle.decompose(oracle.Graph(*args), 2, 1000)
        compare(mp.mpld_decompose(ctx, mp.Graph(*args), 2, 1000, SIMPLIFY | TRACE), ref)


def test_faults(ctx):
    import paper_2303_14335_amd as mp
    say("faults in a large graph")
    n, ce, se = clustered(9004, SMALL, 4.0, True, 11)

    def refused(ce, se, what):
        with pytest.raises(mp.MpldError) as e:
            mp.mpld_decompose(ctx, mp.Graph(n, ce, se), 3, 1000)
        assert e.value.code == -1 and what in str(e.value)

    def put(a, i, pair):
        a = a.copy()
        a[i] = pair
        return a

    refused(put(ce, 77, (3, n)), se, "conflict edge 77 has a node id out of range")
    refused(put(ce, 5, (-1, 2)), se, "conflict edge 5 has a node id out of range")
    refused(put(ce, 0, (9, 9)), se, "conflict edge 0 is a self loop")
    refused(put(ce, 10, ce[900][::-1]), se, "duplicate conflict edge")
    refused(ce, put(se, 3, (n, 0)), "stitch edge 3 is out of range")
    refused(ce, put(se, 4, (se[9][1], se[9][1])), "or a loop")
    refused(ce, put(se, 4, (se[9][1], se[4][0])), "two stitch pairs")
    last = np.array([[ce[40][0], ce[40][1]]], np.int32)
    refused(ce, last, "both stitch and conflict")
    ref = oracle.decompose(oracle.Graph(n, ce, se), 3, 1000)   # and the graph itself still goes through
    compare(mp.mpld_decompose(ctx, mp.Graph(n, ce, se), 3, 1000, SIMPLIFY | TRACE), ref)


def line(n, near, seed):
    """Nodes in a row, each in conflict with `near` on either side; seed 0: ids
    along the row."""
    ids = np.random.default_rng(seed).permutation(n) if seed else np.arange(n)
    ce = np.concatenate([np.stack([ids[:-d], ids[d:]], 1) for d in range(1, near + 1)]).astype(np.int32)
    se = np.stack([ids[0:n - 9:9], ids[5:n - 4:9]], 1).astype(np.int32) if near < 5 else np.zeros((0, 2), np.int32)
    return n, ce, se


def window(rects, aspect):
    """A packed window, cut into `aspect` strips that are laid end to end."""
    side = int(1000 * (rects / 277.0) ** 0.5)
    r = workload.generate(rects, side, 21)[0].copy()
    h = side // aspect
    strip = np.minimum(r[:, 1] // h, aspect - 1)
    r[:, [0, 2]] += (strip * side)[:, None].astype(r.dtype)
    r[:, [1, 3]] -= (strip * h)[:, None].astype(r.dtype)
    g = oracle.build_graph(r, 100, 0)
    return g.num_nodes, g.ce, g.se


# levels, rounds, and whether the host has to take the split or the recovery back
@pytest.mark.parametrize("limits,taken", [((-1, -1), None), ((1 << 20, 1 << 20), (0, 0)), ((0, -1), (1, 0)),
                                          ((1 << 20, 0), (0, 1))])
@pytest.mark.parametrize("shape,k,flags", [
    ("line", 3, SIMPLIFY | TRACE), ("shuffled", 3, SIMPLIFY | TRACE | STITCH), ("shuffled", 3, TRACE),
    ("window", 3, SIMPLIFY | TRACE), ("window", 20, SIMPLIFY | TRACE), ("clusters", 3, SIMPLIFY | TRACE | MARK),
    ("dense", 3, SIMPLIFY | TRACE)])
def test_depth(ctx, shape, k, flags, limits, taken):
    """Deep peelings, long components and long lists, each given up by the
    device where it may not take so many levels, and done there where it may."""
    import paper_2303_14335_amd as mp
    from paper_2303_14335_amd import _ffi
    aspect, k = (k, 3) if shape == "window" else (1, k)
    n, ce, se = {"line": lambda: line(1500, 2, 0), "shuffled": lambda: line(3001, 2, 5),
                 "window": lambda: window(1500, aspect), "dense": lambda: line(700, 90, 4),
                 "clusters": lambda: clustered(3000, [600, 513, 100, 70, 30, 9], 4.6, True, 8)}[shape]()
    say("depth", shape, k, flags, limits)
    left = (ctypes.c_int64 * 2)()
    set_limits = _ffi.load().mpld_test_flow_limits

    def limit(levels, rounds, start):
        assert set_limits(ctx.handle, ctypes.c_int32(levels), ctypes.c_int32(rounds),
                          ctypes.c_int64(start), left) == 0
        return left[0], left[1]

    ref = oracle.decompose(oracle.Graph(n, ce, se), k, 300, bool(flags & SIMPLIFY), bool(flags & MARK),
                           bool(flags & STITCH))
    before = limit(*limits, 1)
    try:
        b = mp.Batch(ctx, mp.Graph(n, ce, se), k, 300, flags)
        for _ in range(2):
            b.solve()
            compare(b.result(), ref)
        b.close()
    finally:
        after = limit(-1, -1, -1)
    if taken is not None:
        removed = int((ref.comp_of < 0).sum())
        deep = shape in ("line", "shuffled") and flags & SIMPLIFY or len(ref.comps) and ref.comps["size"].max() > 64
        # one recovery at most: the batch is the host's from then on
        want = (int(bool(deep)) if taken[0] else 0, int(removed > 0) if taken[1] else 0)
        assert (after[0] - before[0], after[1] - before[1]) == want


@pytest.mark.parametrize("mib", [0, 1, 2, 4, 8, 64])
def test_little_memory(monkeypatch, mib):
    """A graph that the device has no memory for is the host's: the same
    answers with any amount that the components fit in, and a call that was
    refused leaves nothing behind that a later one takes for memory."""
    import torch

    import paper_2303_14335_amd as mp
    say("little memory", mib)
    n, ce, se = clustered(20000, MIXED, 4.4, True, 77)
    args = (mp.Graph(n, ce, se), 3, 300, SIMPLIFY | TRACE)
    ref = oracle.decompose(oracle.Graph(n, ce, se), 3, 300)
    empty, taken = torch.empty, []

    def limited(size, *a, **kw):
        if sum(t.numel() for t in ctx._alloc.live.values()) + size > mib << 20:
            raise torch.OutOfMemoryError("limited")
        taken.append(size)
        return empty(size, *a, **kw)

    ctx = mp.Context(0)
    monkeypatch.setattr(torch, "empty", limited)
    if mib == 0:
        with pytest.raises(mp.MpldError) as e:
            mp.mpld_decompose(ctx, *args)
        assert e.value.code == -2
    else:
        b = mp.Batch(ctx, *args)
        for _ in range(2):   # (without the heavy-component engine's own 96 MiB)
            b.solve()
            compare(b.result(), ref)
        b.close()
    monkeypatch.undo()
    compare(mp.mpld_decompose(ctx, *args), ref)
    ctx.close()
