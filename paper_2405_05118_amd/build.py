"""Builds libmdh.so (the C-ABI library with the HIP kernels) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libmdh.so")

SOURCES = [
    "mdh_plan.cpp",
    "mdh_plan_reduce.cpp",
    "mdh_plan_ex.cpp",
    "mdh_plan_scan.cpp",
    "mdh_plan_capsule.cpp",
    "mdh_plan_split.cpp",
    "mdh_custom.cpp",
    "mdh_api.hip",
    "mdh_stencil.hip",
    "mdh_matmul.hip",
    "mdh_matmul_ksplit.hip",
    "mdh_matmul_split.hip",
    "mdh_matmul_split_k.hip",
    "mdh_mcc.hip",
    "mdh_mcc_split.hip",
    "mdh_mcc_flat.hip",
    "mdh_mcc_flat_split.hip",
    "mdh_calib.hip",
    "mdh_scan.hip",
    "mdh_capsule.hip",
    "mdh_matmul_skinny.hip",
    "mdh_custom_reduce.hip",
    "mdh_custom_reduce_bits.hip",
    "mdh_reduce.hip",
    "mdh_matmul_ex.hip",
]

# packed-fp32 VALU instructions (v_pk_*_f32) are switched off on purpose: some of their forms have
# given wrong results on this hardware; hipcc's host pass prints a harmless "unknown feature" note
HIP_FLAGS = [
    "-O3",
    "-std=c++17",
    "--offload-arch=gfx950",
    "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def build_library(verbose: bool = False, jobs: int = 6) -> str:
    """Compile every source to an object (in parallel) and link libmdh.so.  Always compiles."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    procs = []
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        objs.append(obj)
        cmd = ["hipcc", "-x", "hip", *HIP_FLAGS, *inc, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        while sum(p.poll() is None for _, p in procs) >= jobs:
            for _, p in procs:
                if p.poll() is None:
                    p.wait()
                    break
    failed = False
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(ln for ln in out.splitlines() if "packed-fp32-ops" not in ln)
        if p.returncode != 0:
            failed = True
            sys.stderr.write("hipcc failed on %s:\n%s\n" % (src, out))
        elif verbose and out.strip():
            print(out)
    if failed:
        raise RuntimeError("libmdh build failed")
    tmp = LIB + ".%d.tmp" % os.getpid()
    subprocess.check_call(["hipcc", "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs, "-lhiprtc"])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
