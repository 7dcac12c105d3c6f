"""Compile libpncg.so (HIP, gfx950) in-tree.

    python -m paper_2405_08001_amd.build

Every source under csrc/ is compiled with hipcc for gfx950 (side by side,
into a temporary folder) and linked into paper_2405_08001_amd/libpncg.so.
Packed-FP32 instruction selection is disabled (-packed-fp32-ops) and
float64/float32 global atomics are emitted as hardware atomics
(-munsafe-fp-atomics).  The persistent kernels are compiled without
machine-level loop-invariant code motion: their loops hold a whole iteration,
and the constants and addresses hoisted out cost the step kernel 30 to 70 vector
registers of the 128 (without: 62-127 and no spill but in the contact forms,
which spill up to 4 in float and 22 in double).
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpncg.so")
ARCH = os.environ.get("PNCG_OFFLOAD_ARCH", "gfx950")


def hipcc():
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def flags():
    return ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC",
            "-munsafe-fp-atomics", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wno-unused-result", "-I" + os.path.join(HERE, "..", "include")]


EXTRA_FLAGS = {name: ["-mllvm", "-disable-machine-licm"] for name in ("persist.hip", "adjoint_persist.hip")}


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    # hipcc's host pass warns about the unknown packed-fp32 feature; that is harmless
    msgs = [ln for ln in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in ln]
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs))


def build(verbose=False):
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in srcs]

        def compile_one(src, obj):
            _run([hipcc()] + flags() + EXTRA_FLAGS.get(os.path.basename(src), []) + ["-c", "-o", obj, src], verbose)

        with ThreadPoolExecutor(max_workers=min(len(srcs), 8)) as pool:
            for f in [pool.submit(compile_one, s, o) for s, o in zip(srcs, objs)]:
                f.result()
        out = LIB + ".tmp"
        _run([hipcc(), "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", out] + objs, verbose)
    os.replace(out, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
