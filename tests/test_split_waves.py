"""The device's simplification and split on the CPU, lane by lane, against the
host's: the workgroups that number the largest components run side by side,
and one of them is held up while the others run out of patience."""
import subprocess

import pytest

import simt

# as many workgroups as run side by side here, and patience for minutes or for
# less than a held-up workgroup takes
BLOCKS = ("graph_device.hip", "constexpr int kGiantBlocks = 128;", "constexpr int kGiantBlocks = 4;")
PATIENT = ("graph_device.hip", "kMeetSpin = 1 << 22;", "kMeetSpin = 1 << 30;")
IMPATIENT = ("graph_device.hip", "kMeetSpin = 1 << 22;", "kMeetSpin = 1000000;")
# (the lanes of a wave leave this loop together: the stand-in has no loops of
# different lengths within a wave)
LOOP = ("graph_device.hip", "for (int32_t t = t0, ch = 0; t < t1; t += G, ch += G) {\n    const bool h",
        "for (int32_t t = t0, ch = 0; __ballot(t < t1) != 0; t += G, ch += G) {\n    const bool h")


@pytest.fixture(scope="module")
def exes(tmp_path_factory):
    made = {}

    def get(*edits):
        if edits not in made:
            made[edits] = simt.build(tmp_path_factory.mktemp("split"), "simt_split.cpp", [BLOCKS, LOOP, *edits],
                                     ["frontend.cpp"])
        return made[edits]
    return get


def run(exe, shape, n, k, simplify, seed, hold=-1, levels=1 << 20, more=()):
    out = subprocess.run([exe, shape, str(n), str(k), str(int(simplify)), str(seed), str(hold), str(levels),
                          *map(str, more)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    return out.stdout.strip()


@pytest.mark.parametrize("shape,n,k,simplify,seed", [
    ("random", 3000, 3, True, 1), ("random", 3001, 2, True, 2), ("random", 700, 3, False, 3),
    ("grid", 2500, 2, True, 4), ("grid", 900, 3, False, 5), ("strip", 1200, 2, True, 6), ("line", 600, 3, False, 7)])
def test_equals_the_host(exes, shape, n, k, simplify, seed):
    assert run(exes(PATIENT), shape, n, k, simplify, seed) == "same"


@pytest.mark.parametrize("hold", [0, 1, 2, 6, 7, 20])
def test_a_workgroup_held_up(exes, hold):
    """Whatever the others do meanwhile, the launch ends, with a right split
    or with none."""
    assert run(exes(IMPATIENT), "grid", 2500, 2, False, 8, hold) == "given up"


@pytest.mark.parametrize("shape,n,k,simplify,levels,answer", [
    ("line", 1500, 3, True, -1, "given up"), ("line", 1500, 3, True, 1000, "same"),
    ("line", 1500, 3, True, 100, "given up"), ("strip", 2000, 2, False, 400, "given up"),
    ("strip", 2000, 2, False, -1, "given up"), ("strip", 400, 2, False, 60, "given up"),
    ("strip", 400, 2, False, 200, "same"), ("grid", 2500, 2, False, 40, "given up"),
    ("random", 3000, 3, True, 0, "given up"), ("random", 300, 8, True, 0, "same")])
def test_levels_are_bounded(exes, shape, n, k, simplify, levels, answer):
    """A peeling or a numbering of more levels than it is allowed is left to
    the host."""
    assert run(exes(PATIENT), shape, n, k, simplify, 9 if shape == "random" else 0, levels=levels) == answer


@pytest.mark.parametrize("launch", [3, 14, 15, 16])
def test_after_a_failed_launch(exes, launch):
    """A launch that failed has taken none of the tickets that it was given."""
    assert run(exes(PATIENT), "random", 5000, 3, True, 10, more=[launch]) == "same"
