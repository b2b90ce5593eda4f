"""Builds the gfx950 HIP library ``liblbmadj.so`` in place with hipcc.

Flags: ``-O3`` with IEEE float division/sqrt (no fast-math), ``-fPIC -shared``,
``-Xclang -target-feature -Xclang -packed-fp32-ops`` (packed FP32 VALU
instructions are turned off for all device code) and ``-ffp-contract=on``:
a multiply is fused into an add only inside one source expression, so the
fusion pattern is a property of the source, not of how a node function was
inlined.  The single-context and batched kernels share the node functions,
and with this flag they round identically (batched results are bitwise the
single-context ones).  The library links the profiler's marker library
(rocprofiler-sdk-roctx) for its named ranges.
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbmadj.so")
SOURCES = [os.path.join(CSRC, f) for f in ("lbm_adj.hip", "variants.hip")]
DEPS = SOURCES + [os.path.join(CSRC, f) for f in ("kernels.hpp", "lattice.hpp", "tiles.hpp", "context.hpp", "ops.hpp")] + [
    os.path.join(ROOT, "include", "lbm_adj.h")]
# (Q, QS, variant mask) of the kernels; each is compiled for both precisions in
# a translation unit of its own, so that the build runs in parallel
VARIANTS = [(9, 0, "0"), (9, 5, "0"), (9, 5, "lbmk::kVarVD"), (19, 0, "0"), (19, 0, "lbmk::kVarMRT"), (19, 7, "0"),
            (19, 7, "lbmk::kVarVD"), (19, 7, "lbmk::kVarMRT"), (19, 7, "(lbmk::kVarMRT | lbmk::kVarVD)")]
ARCH = os.environ.get("LBM_OFFLOAD_ARCH", "gfx950")
# profiler marker library (named ranges around forward, recompute and adjoint segments)
ROCM_LIB = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "lib")


def hipcc() -> str:
    for cand in (os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "bin", "hipcc"), "hipcc"):
        if os.path.sep not in cand or os.path.exists(cand):
            return cand
    return "hipcc"


def units() -> list:
    """(source, defines) of every translation unit, the slowest to compile first."""
    out = [(SOURCES[1], ["-DLBM_INSTANTIATE_Q=%d" % q, "-DLBM_INSTANTIATE_QS=%d" % qs,
                         "-DLBM_INSTANTIATE_REAL=%s" % real, "-DLBM_INSTANTIATE_V=%s" % v])
           for q, qs, v in reversed(VARIANTS) for real in ("float", "double")]
    return out + [(SOURCES[0], [])]


def compile_command(src: str, defines, out: str, extra=()) -> list:
    return [hipcc(), "--offload-arch=%s" % ARCH, "-O3", "-std=c++17", "-fPIC",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-ffp-contract=on",
            "-Wall", "-Wno-unused-result", "-I", os.path.join(ROOT, "include"), *defines, *extra, "-c", src, "-o", out]


def link_command(objects, out: str) -> list:
    return [hipcc(), "--offload-arch=%s" % ARCH, "-fPIC", "-shared", "-o", out, *objects, "-L", ROCM_LIB,
            "-Wl,-rpath," + ROCM_LIB, "-lrocprofiler-sdk-roctx"]


def _run(cmd) -> str:
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + proc.stdout + proc.stderr)
    return proc.stderr


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(d) > t for d in DEPS)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile the library (always when force, else only if missing or stale)."""
    if not force and not stale():
        return LIB
    tmp = LIB + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory(prefix="lbmadj_") as work, \
            concurrent.futures.ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
        jobs = [(compile_command(src, defs, os.path.join(work, "%d.o" % i)), os.path.join(work, "%d.o" % i))
                for i, (src, defs) in enumerate(units())]
        notes = list(pool.map(_run, [cmd for cmd, _ in jobs]))
        notes.append(_run(link_command([o for _, o in jobs], tmp)))
    if verbose:
        print("".join(notes))
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
