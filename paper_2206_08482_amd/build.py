"""Builds libgmidrl.so (HIP, gfx950 only) in-tree with hipcc.  `python -m paper_2206_08482_amd.build`."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(HERE, "_build")
LIB_PATH = os.path.join(HERE, "libgmidrl.so")
# the slowest compiles first, so that they overlap all the others
SOURCES = ["fused.hip", "fp8.hip", "agent.hip", "mlp.hip", "tile_p0.hip", "tile_p1.hip", "tile_p2.hip", "tile_p3.hip", "tile_p4.hip", "tile_p5.hip", "tile_f0.hip", "tile_f1.hip", "tile_f2.hip", "tile_f3.hip", "tile_f4.hip", "tile_f5.hip", "tile_q0.hip", "tile_q1.hip", "tile_q2.hip", "tile_q3.hip", "tile_q4.hip",
           "core.hip", "env.hip", "experience.hip", "model.hip", "update.hip", "peaks.hip", "select.hip", "channels.hip", "chain.hip", "f32.hip", "resident.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Wno-unused-value", "-Wno-unused-result", "-fhip-fp32-correctly-rounded-divide-sqrt",
         # keep fp32 arithmetic scalar: packed fp32 forms are not trusted on the test machines
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc(), *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    print(f"compiled {src}", flush=True)
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=8) as pool:
        objs = list(pool.map(_compile, SOURCES))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB_PATH, *objs]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("link failed:\n" + res.stderr)
    if verbose:
        print(f"built {LIB_PATH}")
    return LIB_PATH


if __name__ == "__main__":
    build()
