"""Builds libmpld.so (host C++ and HIP sources for gfx950) in place."""
from __future__ import annotations

import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmpld.so")

SOURCES = ["frontend.cpp", "context.cpp", "runtime.cpp", "abi.cpp", "serve.cpp", "serve_core.cpp", "autotune.cpp", "search_reg.hip",
           "search_lds.hip", "search_device.hip", "graph_device.hip", "flow_device.hip", "seq_engine.hip", "search_min.hip",
           "noalloc.hip", "measure.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# -packed-fp32-ops: never emit packed fp32 ALU ops in device code.
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
          "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", CSRC]


# Per-source flags.  The register tier's search loop branches only on
# wave-uniform values; leaving those regions unstructurized keeps the
# branches as scalar branches instead of exec-mask flow blocks.
EXTRA = {"search_reg.hip": ["-mllvm", "-structurizecfg-skip-uniform-regions"],
         "search_min.hip": ["-mllvm", "-structurizecfg-skip-uniform-regions"],
         # single-lane LDS atomics (the wide tier's per-depth bits) need no
         # rewrite into one atomic per wave
         "search_lds.hip": ["-mllvm", "-amdgpu-atomic-optimizer-strategy=None"]}


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + COMMON + EXTRA.get(src, [])
    if src.endswith(".hip"):
        cmd += ["-x", "hip"]
    cmd += ["-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compiling {src} failed:\n{res.stderr}")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp] + objs + ["-lpthread"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"linking libmpld.so failed:\n{res.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}")
    return LIB


def clean() -> None:
    shutil.rmtree(BUILD, ignore_errors=True)


if __name__ == "__main__":
    build(verbose=True)
