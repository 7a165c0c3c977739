"""Build libhawkes.so for gfx950 in-tree with hipcc (no JIT, no torch extension)."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libhawkes.so")
PEAKS = os.path.join(HERE, "peaks")

# Packed FP32 VALU ops are disabled on purpose: the compiler may form them from
# scalar float code, and the library does not rely on them.
HIPFLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
            "-packed-fp32-ops"]


def _hipcc():
    for c in ("/opt/rocm/bin/hipcc", "hipcc"):
        if os.path.sep not in c or os.path.exists(c):
            return c
    return "hipcc"


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"build failed: {' '.join(cmd)}\n{out}")
    return out


def build_library() -> str:
    """Compiles the sources to objects in parallel (launch.hip once per
    dimension, 1 to 8) and links them."""
    units = [(f, ()) for f in ("hawkes.hip", "serve.hip", "mwg.hip", "hmc.hip", "bmds.hip", "noalloc.hip")]
    units += [("launch.hip", (f"-DHK_D={d}",)) for d in range(1, 9)]
    with tempfile.TemporaryDirectory(prefix="hawkes_build_") as tmpdir:
        objs = [os.path.join(tmpdir, f"{i}.o") for i in range(len(units))]

        def compile_one(i):
            src, defs = units[i]
            _run([_hipcc(), *HIPFLAGS, *defs, "-fPIC", "-c", os.path.join(CSRC, src), "-o", objs[i]])

        # the longest compilations first
        order = sorted(range(len(units)), key=lambda i: units[i][0] not in ("bmds.hip", "launch.hip"))
        with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(compile_one, order))
        tmp = LIB + ".tmp"
        _run([_hipcc(), "--offload-arch=gfx950", "-shared", "-lpthread", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


def build_peaks() -> str:
    _run([_hipcc(), *HIPFLAGS, os.path.join(CSRC, "peaks.hip"), "-o", PEAKS])
    return PEAKS


def build_all() -> None:
    build_library()
    build_peaks()


if __name__ == "__main__":
    build_all()
    print(LIB)
