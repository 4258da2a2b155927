"""Compile the native pieces of the package in-tree.

Two shared libraries live beside this file once built:

* ``libdagsched.so``          - HIP kernels for gfx950 plus the C-ABI (csrc/dagsched.hip)
* ``libdagsched_workload.so`` - seeded synthetic candidate generator (csrc/workload_gen.c)

Nothing here is executed on import; ``ensure_*`` build when the library is absent or older than
its sources, ``build_*`` always recompile.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG_DIR), "include")

HIP_LIB = os.path.join(PKG_DIR, "libdagsched.so")
GEN_LIB = os.path.join(PKG_DIR, "libdagsched_workload.so")

# The host code with most kernels, and the instantiations of the ring kernel: (cell format, lanes per machine) a unit.
RING_UNITS = [(0, 1), (1, 1), (2, 1), (3, 1), (4, 1), (5, 1), (0, 2), (2, 2), (0, 4), (2, 4)]
HIP_UNITS = [("dagsched.hip", [])] + [("ring_kernels.hip", ["-DDAGSCHED_RING_HALF=%d" % h, "-DDAGSCHED_RING_SUB=%d" % s]) for h, s in RING_UNITS]
HIP_FLAGS = ["--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-function", "-I", INCLUDE]


def _run(cmd):
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError("build failed: %s\n%s" % (" ".join(cmd), proc.stdout))
    return proc.stdout


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found; the HIP library cannot be built")


def build_hip(verbose: bool = False) -> str:
    """hipcc -> libdagsched.so (gfx950 only); the units are compiled side by side."""
    tmp = HIP_LIB + ".tmp"
    with tempfile.TemporaryDirectory(prefix="dagsched_build_") as where, ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
        objects = [os.path.join(where, "%d.o" % i) for i in range(len(HIP_UNITS))]
        jobs = [pool.submit(_run, [_hipcc(), *HIP_FLAGS, "-O3", "-fPIC", "-Wall", *defines, "-c", os.path.join(CSRC, source), "-o", obj])
                for obj, (source, defines) in zip(objects, HIP_UNITS)]
        out = "".join(j.result() for j in jobs)
        out += _run([_hipcc(), "--offload-arch=gfx950", "-fPIC", "-shared", *objects, "-o", tmp])
    os.replace(tmp, HIP_LIB)
    if verbose and out.strip():
        print(out)
    return HIP_LIB


def build_workload_gen() -> str:
    """gcc -> libdagsched_workload.so (host only)."""
    tmp = GEN_LIB + ".tmp"
    _run(["gcc", "-O2", "-std=c11", "-fPIC", "-shared", "-Wall",
          os.path.join(CSRC, "workload_gen.c"), "-o", tmp])
    os.replace(tmp, GEN_LIB)
    return GEN_LIB


def _stale(lib: str, sources) -> bool:
    if not os.path.exists(lib):
        return True
    t = os.path.getmtime(lib)
    return any(os.path.exists(s) and os.path.getmtime(s) > t for s in sources)


def ensure_workload_gen() -> str:
    if _stale(GEN_LIB, [os.path.join(CSRC, "workload_gen.c")]):
        build_workload_gen()
    return GEN_LIB


def hip_sources():
    """Every file the HIP library is compiled from: the kernels, the host code and the public header."""
    import glob
    return sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip")) +
                  glob.glob(os.path.join(INCLUDE, "*.h")))


def ensure_hip() -> str:
    """Return the built HIP library; compile it when it is absent or older than one of its sources (where no
    compiler is at hand, as on a box that only runs what was built elsewhere, a stale library is an error)."""
    if _stale(HIP_LIB, hip_sources()):
        build_hip()
    return HIP_LIB
