"""The sequence engine's workspace, on the CPU with stand-ins for the searches:
nothing is given back while launches that use it are on the way, and a pool
that has not as much is no error."""
import subprocess

import pytest

import simt


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return simt.build(tmp_path_factory.mktemp("seq"), "simt_seq.cpp", also=["context.cpp"])


@pytest.mark.parametrize("mib,least,most", [(0, 0, 0), (1, 0, 0), (40, 1, 8), (300, 4, 8), (4096, 8, 8)])
def test_workspace(exe, mib, least, most):
    out = subprocess.run([exe, str(mib)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, (out.stdout, out.stderr)
    assert least <= int(out.stdout) <= most


@pytest.fixture(scope="module")
def room(tmp_path_factory):
    return simt.build(tmp_path_factory.mktemp("room"), "simt_room.cpp")


@pytest.mark.parametrize("tasks,arena", [(2000, 1 << 20), (1 << 20, 1 << 18), (3000, 1 << 18), (24, 64)])
def test_refused_requests_take_nothing(room, tasks, arena):
    """Each place is given once, and the counts stand still once there is no
    room, however often it is asked for."""
    out = subprocess.run([room, str(tasks), str(arena), "7"], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, (out.stdout, out.stderr)
