"""Builds libkeep_hip.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python -m paper_2602_23592_amd.build
"""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libkeep_hip.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-result", "-Wno-unknown-warning-option",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


# Kernels that must not use scratch memory at all.  k_gemm_256: its accumulators are written by inline assembly, and a spill
# of one right behind a product would store a stale value.  k_gemm_stream: one wave per SIMD hides nothing behind a spill
# (gate/up of 5120 x 55296 with 24 spilled registers: 107 us, 97 without).
NO_SCRATCH = {"gemm_mfma.hip": "k_gemm_256", "gemm_stream.hip": "k_gemm_stream"}


def check_scratch(src, report):
    if src not in NO_SCRATCH:
        return
    kernel, seen = None, 0
    for line in report.splitlines():
        name = re.search(r"Function Name: (\S+)", line)
        if name:
            kernel = name.group(1)
        size = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if size and kernel and NO_SCRATCH[src] in kernel:
            seen += 1
            if int(size.group(1)):
                raise RuntimeError("%s uses %s bytes of scratch memory per lane; it must use none" % (kernel, size.group(1)))
    if not seen:
        raise RuntimeError("no resource report for %s in %s" % (NO_SCRATCH[src], src))


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def build(verbose: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    objs = []

    def compile_one(src):
        obj = os.path.join(OBJ, src[:-4] + ".o")
        report = ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics"] if src in NO_SCRATCH else []
        cmd = [HIPCC, *FLAGS, *report, "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
        check_scratch(src, r.stderr)
        if verbose:
            errs = [l for l in r.stderr.splitlines()
                    if "packed-fp32-ops" not in l and "kernel-resource-usage" not in l and l.strip()]
            print("compiled", src, ("\n" + "\n".join(errs)) if errs else "", flush=True)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(compile_one, sources()))
    cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    if verbose:
        print("linked", LIB, flush=True)
    return LIB


if __name__ == "__main__":
    build()
    sys.exit(0)
