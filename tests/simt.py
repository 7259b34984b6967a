"""Builds a kernel's source for the CPU (tests/native/simt): lanes as fibers,
so that waves and workgroups meet in many orders."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2303_14335_amd", "csrc")
NATIVE = os.path.join(ROOT, "tests", "native")
# a select by a lane mask, the one instruction written as assembly
SELECT = 'asm("v_cndmask_b32_e64 %0, 0, %1, %2" : "=v"(r) : "v"(x), "s"(mask));'


def build(folder, driver, edits=(), also=()):
    """The driver over a copy of the kernels' sources in `folder`; edits:
    (file, text, other text), each there exactly once; also: host sources."""
    gxx = shutil.which("g++")
    if gxx is None or os.uname().machine != "x86_64":
        pytest.skip("needs g++ on x86-64")
    src = os.path.join(str(folder), "csrc")
    os.makedirs(src)
    for f in os.listdir(CSRC):
        if f.endswith((".h", ".hip", ".inc")):
            shutil.copy(os.path.join(CSRC, f), src)
    for name, text, other in (("min_core.h", SELECT, "r = (mask >> __lane_id()) & 1u ? x : 0u;"), *edits):
        path = os.path.join(src, name)
        with open(path) as f:
            s = f.read()
        assert s.count(text) == 1, (name, text)
        with open(path, "w") as f:
            f.write(s.replace(text, other))
    exe = os.path.join(str(folder), "run")
    done = subprocess.run([gxx, "-x", "c++", "-std=c++17", "-O2", "-w", "-I", os.path.join(NATIVE, "simt"), "-I", src,
                           "-I", os.path.join(ROOT, "include"), os.path.join(NATIVE, driver),
                           *(os.path.join(CSRC, f) for f in also), "-o", exe, "-lpthread"],
                          capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    return exe
