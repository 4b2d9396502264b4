"""Builds libkeep_hip.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree.

    python -m paper_2602_23592_amd.build
"""
import os
import re
import subprocess
import sys
import tempfile
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


# Kernels that keep their accumulators in accumulation registers by inline assembly: the compiler does not know when a product
# is finished, so a copy of its own making (a move behind a product) would read a stale value.
ASM_ACCUMULATORS = {"gemm_mfma.hip": "k_gemm_256"}


def check_accumulators(src, assembly):
    """No instruction outside the inline assembly of such a kernel touches an accumulation register."""
    seen = 0
    for name, body in re.findall(r"^(_Z\w*%s\w*):[^\n]*\n(.*?)^\.Lfunc_end" % ASM_ACCUMULATORS[src], assembly, re.S | re.M):
        seen += 1
        ours = False
        for line in body.splitlines():
            if "#ASMSTART" in line or "#ASMEND" in line:
                ours = "#ASMSTART" in line
            elif not ours and re.search(r"\ba(\d+|\[\d+)", line.split(";")[0]):
                raise RuntimeError("%s: the compiler touches an accumulator: %s" % (name, line.strip()))
    if not seen:
        raise RuntimeError("no assembly of %s in %s" % (ASM_ACCUMULATORS[src], src))


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def build(verbose: bool = True, jobs: int = 8) -> str:
    os.makedirs(OBJ, exist_ok=True)
    objs = []

    def compile_one(src):
        obj = os.path.join(OBJ, src[:-4] + ".o")
        report = ["-Rpass-analysis=kernel-resource-usage", "-fno-caret-diagnostics"] if src in NO_SCRATCH else []
        with tempfile.TemporaryDirectory(dir=OBJ) as tmp:
            made = os.path.join(tmp, os.path.basename(obj))
            temps = ["-save-temps=obj", "-Wno-tautological-compare"] if src in ASM_ACCUMULATORS else []
            r = subprocess.run([HIPCC, *FLAGS, *report, *temps, "-c", os.path.join(CSRC, src), "-o", made],
                               capture_output=True, text=True)
            if r.returncode != 0:
                raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
            check_scratch(src, r.stderr)
            if temps:
                asm, = (f for f in os.listdir(tmp) if f.endswith(".s") and "amdgcn" in f)
                with open(os.path.join(tmp, asm)) as f:
                    check_accumulators(src, f.read())
            os.replace(made, obj)
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
