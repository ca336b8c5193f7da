"""Builds the HIP library libot_assoc.so for gfx950 in-tree with hipcc."""

from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libot_assoc.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    # keep hipcc from forming packed FP32 instructions on its own
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result",
]


def sources():
    return [os.path.join(CSRC, f) for f in ("ot_assoc.hip", "launch_dense.hip", "launch_rates.hip", "launch_geo.hip",
                                            "coop_dense.hip", "coop_dense64.hip", "coop_rates.hip", "coop_geo.hip",
                                            "batch.hip", "team.hip", "snapshots.hip")]


def _compile(src: str, obj: str, inc: str):
    cmd = [HIPCC, *FLAGS, "-c", "-I", inc, "-o", obj, src]
    return cmd, subprocess.run(cmd, capture_output=True, text=True)


def build(verbose: bool = False) -> str:
    """Compile every HIP source of the library (one process per source) and
    link libot_assoc.so; always rebuilds."""
    from concurrent.futures import ThreadPoolExecutor

    inc = os.path.join(os.path.dirname(HERE), "include")
    bdir = os.path.join(HERE, "_build")
    os.makedirs(bdir, exist_ok=True)
    srcs = sources()
    objs = [os.path.join(bdir, os.path.basename(s) + ".o") for s in srcs]
    with ThreadPoolExecutor(max_workers=len(srcs)) as ex:
        results = list(ex.map(lambda so: _compile(so[0], so[1], inc), zip(srcs, objs)))
    for cmd, r in results:
        if verbose:
            print(" ".join(cmd), flush=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError("hipcc failed building libot_assoc.so")
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("linking libot_assoc.so failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
