"""Builds liblenia.so (HIP, gfx950) in-tree with hipcc.

Every HIP/C++ source under csrc/ is compiled to an object in _build/ (in
parallel) and linked into paper_2304_05639_amd/liblenia.so.  Packed-FP32
instructions are disabled for all device code, and a kernel that the compiler
gives accumulation registers (AGPRs) fails the build: with a budget of 512
registers (one wave per SIMD) it split a value's life between the two files
inside divergent branches of the four-cell step kernel, and results were wrong.
Launch bounds that leave at most 256 registers keep every kernel off them.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblenia.so")
ARCH = os.environ.get("LENIA_OFFLOAD_ARCH", "gfx950")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
          f"--offload-arch={ARCH}", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
          "-fvisibility=hidden", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Rpass-analysis=kernel-resource-usage"]


def split_remarks(stderr: str):
    """(AGPRs by kernel, the other lines) of hipcc's output with resource remarks,
    each of which may be followed by the source line it points at."""
    agprs, rest, kernel, remark = {}, [], None, False
    for line in stderr.splitlines():
        if "-Rpass-analysis=kernel-resource-usage" in line:
            m = re.search(r"remark:\s+(Function Name|AGPRs): (\S+)", line)
            if m and m[1] == "AGPRs":
                agprs[kernel] = int(m[2])
            elif m:
                kernel = m[2]
            remark = True
        elif not (remark and re.match(r"\s*\d* \|", line)):
            remark = False
            rest.append(line)
    return agprs, "\n".join(rest)


def check_registers(agprs) -> None:
    used = {k: n for k, n in agprs.items() if n}
    if used:
        raise RuntimeError(f"kernels with accumulation registers: {used}; tighten their launch bounds")


def _compile(src: str) -> str:
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    lang = ["-x", "hip"]
    cmd = [HIPCC] + COMMON + lang + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    agprs, err = split_remarks(r.stderr)
    err = "\n".join(l for l in err.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{err}")
    check_registers(agprs)
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(jobs: int = 8) -> str:
    os.makedirs(BUILD, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))
    with cf.ThreadPoolExecutor(max_workers=min(jobs, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build())
