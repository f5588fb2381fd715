"""Builds the HIP libraries in-tree for gfx950: ``libphub.so`` (the
exchange step and its C interface) and ``libphub_probe.so`` (the bandwidth
probe that the benchmark times beside the step) and ``libphub_roots.so`` (a
check of the device's square roots).

Every source is compiled by hipcc with contraction off, no fast-math,
subnormals kept, and divisions and roots correctly rounded, so that the
kernel performs exactly the fp32 operations the step defines; packed fp32
instructions are disabled.
"""

from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile
from typing import Sequence

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libphub.so")
PROBE_LIB = os.path.join(PKG, "libphub_probe.so")
# Ablation build: the gradients loaded cache-allocating (run it with
# bench.py --library); not built by default.
GRADIENTS_CACHED_LIB = os.path.join(PKG, "libphub_gradients_cached.so")
PROBE_SOURCES = ["probe.hip"]
ROOTS_LIB = os.path.join(PKG, "libphub_roots.so")
ROOTS_SOURCES = ["roots.hip"]

SOURCES = ["plan.cpp", "phub_api.cpp", "fused_step.hip", "fused_stream.hip", "fused_many.hip",
           "fused_many_shared.hip", "put_pointers.hip", "step_noalloc.hip"]
HEADERS = ["plan.hpp", "kernels.hpp", "device.hpp", "tile_walk.hpp", "stream_walk.hpp",
           "many_walk.hpp"]
# Sources that hold many kernels, and the parts (PHUB_STEP_PART) that they are
# compiled in
PARTS = {"fused_step.hip": range(8), "fused_stream.hip": range(0, 8, 2)}

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    "-ffp-contract=off",
    "-fno-fast-math",
    "-fno-gpu-flush-denormals-to-zero",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall",
]


def build(out: str = LIB, defines: Sequence[str] = (), extra: Sequence[str] = (),
          verbose: bool = False) -> str:
    """Compile the sources side by side and link the library; returns its
    path.  ``defines`` are extra -D settings (used for launch-shape sweeps)."""
    flags = [f for f in FLAGS if f != "-shared"]
    units = []  # (source, its own defines), the longest compilations first
    for s in sorted(SOURCES, key=lambda s: s not in PARTS):
        units += [(s, [] if p is None else [f"PHUB_STEP_PART={p}"]) for p in PARTS.get(s, (None,))]
    with tempfile.TemporaryDirectory(dir=os.path.dirname(os.path.abspath(out))) as tmp:
        def compile_one(i: int) -> str:
            src, own = units[i]
            obj = os.path.join(tmp, f"{i}.o")
            cmd = [HIPCC, *flags, f"-I{INCLUDE}", f"-I{CSRC}", *[f"-D{d}" for d in defines],
                   *[f"-D{d}" for d in own], *extra, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return obj

        with concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            objs = list(pool.map(compile_one, range(len(units))))
        lib = os.path.join(tmp, "lib.so")
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", lib])
        os.replace(lib, out)
    return out


def build_probe(out: str = PROBE_LIB, verbose: bool = False,
                sources: Sequence[str] = PROBE_SOURCES) -> str:
    """Compile the bandwidth probe library; returns its path."""
    srcs = [os.path.join(CSRC, s) for s in sources]
    tmp = out + ".tmp"
    cmd = [HIPCC, *FLAGS, f"-I{INCLUDE}", *srcs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, out)
    return out


def device_assembly(out: str, source: str = "fused_step.hip", defines: Sequence[str] = ()) -> str:
    """Compile one HIP source of the library to gfx950 device assembly (with
    its kernel metadata: registers, LDS, scratch, spills) at ``out``; the
    code-generation tests read it.  ``defines`` as ``build``'s."""
    flags = [f for f in FLAGS if f not in ("-fPIC", "-shared")]
    cmd = [HIPCC, *flags, f"-I{INCLUDE}", f"-I{CSRC}", *[f"-D{d}" for d in defines],
           "--cuda-device-only", "-S",
           os.path.join(CSRC, source), "-o", out]
    subprocess.check_call(cmd, stderr=subprocess.DEVNULL)
    return out


def build_all(verbose: bool = False) -> None:
    build(verbose=verbose)
    build_probe(verbose=verbose)
    build_probe(ROOTS_LIB, verbose, ROOTS_SOURCES)


def build_gradients_cached(verbose: bool = False) -> str:
    """The ablation library whose kernels load the gradients
    cache-allocating (PHUB_GRADIENT_LOADS_CACHED) instead of non-temporally."""
    return build(GRADIENTS_CACHED_LIB, defines=["PHUB_GRADIENT_LOADS_CACHED=1"], verbose=verbose)


if __name__ == "__main__":
    if "--gradients-cached" in sys.argv[1:]:
        build_gradients_cached(verbose=True)
    else:
        build_all(verbose=True)
    sys.exit(0)
