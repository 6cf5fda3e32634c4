"""Build the HIP library ``libdvl.so`` (gfx950) in-tree.

    python -m paper_2306_11612_amd.build

Compiles every ``csrc/*.hip`` with hipcc into ``paper_2306_11612_amd/_lib/``,
plus one generated translation unit per (storage type, field count) that
instantiates the typed update kernels (``launch_sm`` in
``csrc/update_kernels.hpp``), so that they compile in parallel.  Packed fp32
instructions are disabled for all device code.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT_DIR = os.path.join(HERE, "_lib")
LIB = os.path.join(OUT_DIR, "libdvl.so")
ARCH = os.environ.get("DVL_OFFLOAD_ARCH", "gfx950")

# Kernels whose inputs are NaN-free by contract (build_order rejects NaN field
# values) drop IEEE NaN handling of min/max, which otherwise doubles every
# fminf/fmaxf with canonicalisations.  Host code keeps full IEEE semantics.
_NO_NAN = ["-Xarch_device", "-fno-honor-nans", "-Xarch_device", "-mno-amdgpu-ieee"]
TYPED_UNITS = [(t, m) for t in ("F32", "F16", "BF16") for m in (1, 2, 3, 4, 5, 6, 7, 8, 16)]
FILE_FLAGS = {"update.hip": _NO_NAN}
FILE_FLAGS.update({f"update_{t.lower()}_m{m}.hip": _NO_NAN for t, m in TYPED_UNITS})


def generated_sources(gen_dir: str) -> list[str]:
    """Write the instantiation units of the typed update kernels (rewritten
    only when their text changes) and return their paths."""
    os.makedirs(gen_dir, exist_ok=True)
    paths = []
    for t, m in TYPED_UNITS:
        path = os.path.join(gen_dir, f"update_{t.lower()}_m{m}.hip")
        text = ("// Generated by paper_2306_11612_amd/build.py: the update kernels for\n"
                f"// {t} storage and {m}-field jobs.\n"
                '#include "update_kernels.hpp"\n\n'
                "namespace dvl {\n"
                f"template dvl_status launch_sm<{t}, {m}>(const BatchLaunch&, int, hipStream_t, uint64_t, hipEvent_t*);\n"
                "}  // namespace dvl\n")
        old = open(path).read() if os.path.exists(path) else None
        if old != text:
            with open(path, "w") as fh:
                fh.write(text)
        paths.append(path)
    return paths

HIPCC_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unused-result",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def build(verbose: bool = False, jobs: int = 0) -> str:
    """Compile all sources (always; object files are rebuilt in parallel) and link."""
    jobs = jobs or max(1, min(16, os.cpu_count() or 1))
    os.makedirs(OUT_DIR, exist_ok=True)
    obj_dir = os.path.join(OUT_DIR, "obj")
    os.makedirs(obj_dir, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip"))) + generated_sources(os.path.join(OUT_DIR, "gen"))
    procs, objs = [], []
    for src in srcs:
        obj = os.path.join(obj_dir, os.path.basename(src) + ".o")
        objs.append(obj)
        cmd = [_hipcc(), *HIPCC_FLAGS, *FILE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            procs[[p.poll() is None for _, p in procs].index(True)][1].wait()
    failed = []
    for src, p in procs:
        out, _ = p.communicate()
        text = out.decode(errors="replace")
        if p.returncode != 0:
            failed.append((src, text))
        elif verbose and text.strip():
            print(text)
    if failed:
        msg = "\n".join(f"--- {s}\n{t}" for s, t in failed)
        raise RuntimeError(f"hipcc failed:\n{msg}")
    tmp = LIB + ".tmp"
    cmd = [_hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    subprocess.check_call(cmd)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
