"""Build libheget.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python paper_0908_4403_amd/build.py [-v]

Every HIP source is compiled with packed-FP32 instructions disabled
(-Xclang -target-feature -Xclang -packed-fp32-ops); hipcc's host pass warns
that it does not know the feature, which is harmless.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libheget.so")
BUILD_DIR = os.path.join(PKG, "_build")

# slowest first, so that the pool starts them at once
SOURCES = ["me2_shapes_f32_meet8.hip", "me2_shapes_sampled_meet8.hip", "me2_shapes_f32_meet7.hip", "me2_shapes_f32_whole.hip",
           "me2_shapes_f32_lo.hip", "me2_shapes_f32_mid.hip", "me2_shapes_f32_hi.hip",
           "me2_shapes_f64_lo.hip", "me2_shapes_f64_mid.hip", "me2_shapes_f64_hi.hip",
           "me2_shapes_sampled.hip", "me2_lanes.hip", "me2_pair.hip", "me2_batch.hip", "me2_registry.cpp", "mc_kernels.hip", "mc_fused.hip", "peak.hip", "helas_kernels.hip",
           "static_scratch.hip",
           "heget_api.cpp"]
ARCH = os.environ.get("HEGET_OFFLOAD_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = [f"--offload-arch={ARCH}", "-O3", "-fPIC", "-std=c++17",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wno-unused-command-line-argument",
          "-I", INCLUDE, "-I", CSRC]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *COMMON, "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    msg = "\n".join(l for l in (r.stderr or "").splitlines()
                    if "not a recognized feature for this target" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{msg}")
    if verbose and msg.strip():
        print(msg, flush=True)
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 4)) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
