"""Build libqcoll.so in-tree with hipcc for gfx950.

    python -m paper_2103_14890_amd.build [--verbose]
"""

from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys
import tempfile

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libqcoll.so")

HOST_SOURCES = ["plan.cpp", "api.cpp", "transport.cpp"]
DEVICE_SOURCES = ["kernels_multi.hip", "kernels_fft.hip", "kernels_fft64.hip", "kernels_2d.hip", "kernels_2d16.hip", "kernels_2d64.hip", "kernels_3d.hip",
                  "kernels_galerkin.hip", "kernels_transport.hip", "kernels_classical.hip", "noalloc.hip"]
ARCH = "gfx950"

COMMON = ["-O3", "-std=c++17", "-fPIC", f"-I{INCLUDE}", f"-I{CSRC}", "-I/opt/rocm/include", "-D__HIP_PLATFORM_AMD__"]
# Packed FP32 VALU instructions are disabled in all device code.
# MFMA accumulators are kept in VGPRs so that VALU code reads them directly.
DEVICE_FLAGS = [f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-ffp-contract=fast", "-mllvm", "-amdgpu-mfma-vgpr-form=1"]
# Per-file additions: the 32x32 kernels are scheduled for instruction-level
# parallelism (3% shorter eval launches at the same register count and bitwise
# equal results; the 64-point kernels were 1.5% slower with it).
# The batched kernel reads its slot table in place: with more reads of it than
# the compiler's default limit (300) the table is copied to each lane's scratch.
FILE_FLAGS = {"kernels_2d.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
              "kernels_multi.hip": ["-mllvm", "-instcombine-max-copied-from-constant-users=100000"]}


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + res.stderr)
        raise RuntimeError(f"build step failed: {' '.join(cmd[:3])} ...")
    if verbose and res.stderr.strip():
        sys.stderr.write(res.stderr)


def build(verbose: bool = False, extra: list[str] | None = None) -> str:
    """Compile every source and link libqcoll.so next to this file. Always rebuilds."""
    hipcc = _hipcc()
    extra = list(extra or [])
    with tempfile.TemporaryDirectory(prefix="qcoll_build_") as tmp:
        cmds, objs = [], []
        for src in HOST_SOURCES:
            obj = os.path.join(tmp, src + ".o")
            cmds.append([hipcc, "-x", "c++", *COMMON, *extra, "-c", os.path.join(CSRC, src), "-o", obj])
            objs.append(obj)
        for src in DEVICE_SOURCES:
            obj = os.path.join(tmp, src + ".o")
            cmds.append([hipcc, "-x", "hip", *COMMON, *DEVICE_FLAGS, *FILE_FLAGS.get(src, []), *extra, "-c",
                         os.path.join(CSRC, src), "-o", obj])
            objs.append(obj)
        # independent compilations, a few at a time
        jobs = max(1, min(8, os.cpu_count() or 1))
        with concurrent.futures.ThreadPoolExecutor(jobs) as ex:
            for fut in [ex.submit(_run, c, verbose) for c in cmds]:
                fut.result()
        tmp_lib = os.path.join(tmp, "libqcoll.so")
        _run([hipcc, "-shared", f"--offload-arch={ARCH}", *objs, "-o", tmp_lib], verbose)
        shutil.copyfile(tmp_lib, LIB + ".tmp")
        os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="--verbose" in sys.argv)
    print(LIB)
