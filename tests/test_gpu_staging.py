"""Batches on both sides of the sizes where a batch's image goes up, and its
results come down, in one staged copy: the answers against the oracle's and
against each other, with other calls on the context between a solve and its
result."""
import numpy as np
import pytest

import oracle
import workload
from algx_literal import random_graph

pytestmark = pytest.mark.gpu

MARK = 1 << 10


def say(*a):
    print("[case]", *a, flush=True)


def components(count, n, seed):
    """Components of n nodes with a few edges each (colored at once)."""
    rng = np.random.default_rng(seed)
    few = [random_graph(rng, n, 2.0 / n) for _ in range(7)]
    return [(n, few[i % 7]) for i in range(count)]


# items of 64 nodes take 560 bytes or so: 256 KiB up hold about 470 of them;
# 88 bytes down each, 256 KiB hold about 2980; 64 KiB of colors are 1024
@pytest.mark.parametrize("count", [1, 455, 460, 465, 470, 475, 480, 1023, 1024, 1025, 2970, 2980, 2990])
@pytest.mark.parametrize("flags", [0, MARK])
def test_sizes_around_the_staging(ctx, count, flags):
    import paper_2303_14335_amd as mp
    comps = components(count, 64, 5)
    say("components", count, "flags", flags)
    a = mp.mpld_solve_components(ctx, comps, 3, 5000, flags)
    b = mp.mpld_solve_components_noalloc(ctx, comps, 3, 5000, flags)
    for f in a[0].dtype.names:
        assert np.array_equal(a[0][f], b[0][f]), f
    assert np.array_equal(np.concatenate(a[1]), np.concatenate(b[1]))
    ref = [oracle.solve_component(n, e, 3, 5000) for n, e in comps[:7]]
    for i in range(count):
        assert a[0]["nodes"][i] == ref[i % 7].nodes and a[0]["status"][i] == ref[i % 7].status
        if ref[i % 7].status == 0:
            assert np.array_equal(a[1][i], ref[i % 7].colors)


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("timed", [False, True])
def test_result_after_other_calls(ctx, split, timed):
    """A batch's result is its last solve's, whatever ran on the context since."""
    import paper_2303_14335_amd as mp
    graphs = [oracle.build_graph(workload.generate(300 + 40 * i, 3160, 60 + i)[0], 100, 0) for i in range(3)]
    refs = [oracle.decompose(g, 3, 2000) for g in graphs]
    say("interleaved batches, split", split, "timed", timed)
    mine = [mp.Graph(g.num_nodes, g.ce, g.se) for g in graphs]
    bs = [mp.Batch(ctx, g, 3, 2000) for g in mine]
    for _ in range(2):
        for b in bs:
            b.solve(split=split, timed=timed)
        other = mp.mpld_decompose(ctx, mine[0], 3, 2000)
        assert np.array_equal(other.colors, refs[0].colors)
        for b, ref in zip(bs, refs):
            for _ in range(2):
                r = b.result()
                assert np.array_equal(r.colors, ref.colors)
                assert np.array_equal(r.components["nodes"], ref.comps["nodes"])
    for b in bs:
        b.close()
