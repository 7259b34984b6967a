"""The kernels of the Eq. 1 minimisation on the CPU, lane by lane, against the
oracle's branch and bound: the waves of a workgroup take and cut pieces in
drawn orders, and with few piece ids, so that cuts find no room and ids are
taken while others give up.  Node counts and colors are the sequential
search's, and every launch ends."""
import subprocess

import numpy as np
import pytest

import oracle
import simt
from algx_literal import random_graph

WAVES = "kMinWaves = 8, kMinItems = 192, kMinPieces = 8"


@pytest.fixture(scope="module")
def exes(tmp_path_factory):
    made = {}

    def get(items, stuck=None):
        if (items, stuck) not in made:
            edits = [("search_min.hip", WAVES, f"kMinWaves = 8, kMinItems = {items}, kMinPieces = 8")]
            if stuck is not None:   # as if round `stuck` had taken no piece off the front
                edits.append(("search_min.hip", "} else if (front == 0) {", f"}} else if (p.round == {stuck}u) {{"))
            made[items, stuck] = simt.build(tmp_path_factory.mktemp("min"), "simt_minimize.cpp", edits)
        return made[items, stuck]
    return get


def component(rng, k):
    n = int(rng.integers(14, 34))
    e = random_graph(rng, n, min(0.95, float(rng.uniform(1.6, 2.4)) * 2.0 * k / n))
    part, perm, es = [-1] * n, rng.permutation(n), {tuple(sorted(p)) for p in e}
    for a, b in perm[: n // 2 * 2].reshape(-1, 2).tolist():
        if rng.random() < 0.5 and tuple(sorted((a, b))) not in es:
            part[a], part[b] = b, a
    return n, e, part


def text(k, budget, seed, comps):
    lines = [f"{k} {budget} {seed} {len(comps)}"]
    for n, e, part, inc in comps:
        nb = [0] * n
        for a, b in e:
            nb[a] |= 1 << b
            nb[b] |= 1 << a
        lines += [str(n), " ".join(map(str, nb)), " ".join(str(p if p >= 0 else 255) for p in part),
                  " ".join(str(int(c)) for c in inc)]
    return "\n".join(lines)


@pytest.mark.parametrize("count", [1, 5, 17, 40, 191])
def test_ids_are_taken_once(exes, count):
    """Eight waves take 1 to 8 ids at a time off one stack, at all points of
    each other's steps."""
    out = subprocess.run([exes(192), "ids", str(count), "3"], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr


@pytest.mark.parametrize("items,k,budget,stuck", [
    (192, 4, 3000, None), (60, 4, 3000, None), (40, 3, 1200, None), (24, 2, 1000, None), (16, 5, 1500, None),
    (12, 4, 65, None), (192, 4, 800, 1), (192, 3, 800, 4)])
def test_pieces(exes, items, k, budget, stuck):
    rng = np.random.default_rng(items * 100 + k)
    comps = []
    while len(comps) < 3:
        n, e, part = component(rng, k)
        inc = oracle.mark_conflicts(n, e, k)
        if abs(oracle.minimize_component(n, e, k, inc, budget, part).nodes) > 64:
            comps.append((n, e, part, inc))
    out = subprocess.run([exes(items, stuck)], input=text(k, budget, items + k, comps), capture_output=True, text=True,
                         timeout=300)
    assert out.returncode == 0, out.stderr
    rows = [list(map(int, line.split())) for line in out.stdout.splitlines()]
    assert len(rows) == len(comps)
    for (n, e, part, inc), row in zip(comps, rows):
        ref = oracle.minimize_component(n, e, k, inc, budget, part)
        assert row[0] == (-ref.nodes if ref.stopped else ref.nodes)
        assert row[1:] == list(ref.colors)
