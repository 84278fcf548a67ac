"""Builds libpf.so (host analysis + gfx950 kernels) in-tree with hipcc."""
from __future__ import annotations

import os
import re
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
BUILD = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libpf.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

ARCH = "gfx950"
# HIP translation units: shared host ABI, Newton path, separate Jacobian and
# factorisation, fast decoupled, state estimation
KERNEL_FILES = ("pf_abi.hip", "pf_newton.hip", "pf_steps.hip", "pf_fdpf.hip", "pf_se.hip")
# Packed fp32 instructions are kept off for every device compile.
DEVICE_FLAGS = ["--offload-arch=" + ARCH, "-Xclang", "-target-feature", "-Xclang",
                "-packed-fp32-ops"]
# The iteration kernels' loops would have the sine's constants hoisted out of
# them, some 30 vector registers for the whole iteration; without that pass the
# fast decoupled kernels (114 to 118 registers, else 128 and spills) keep two
# workgroups per compute unit, and Newton's run 1% faster (200 buses, 487 x 33).
# The other files keep the pass: the factorisation of a band of 500 buses takes
# 6.6 ms with it and 7.2 without, a Jacobian row of 200 entries 58 and 63 us.
FILE_OPT = {f: ["-mllvm", "-disable-machine-licm"] for f in ("pf_newton.hip", "pf_fdpf.hip")}
USAGE = "-Rpass-analysis=kernel-resource-usage"
COMMON = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-I", INCLUDE, "-I", CSRC]


def _no_scratch(lines):
    """Refuses a kernel that uses scratch memory.  The compiler has placed
    the spill of a vector register where only some lanes were active (in the
    join of a branch, before the lanes were enabled again), so that the others
    reloaded garbage; kept in registers the kernels are right, and faster."""
    name = ""
    for line in lines:
        if "Function Name: " in line:
            name = line.split("Function Name: ")[1].split()[0]
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m and int(m.group(1)):
            raise RuntimeError(f"build failed: {name} uses {m.group(1)} bytes of scratch per "
                               "lane; lower its register use")


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines = r.stdout.splitlines()
    if USAGE in cmd:
        _no_scratch(lines)
        # the remarks come with three lines of source each
        cut = [i for i, l in enumerate(lines) if "[-Rpass-analysis" in l]
        drop = {j for i in cut for j in range(i, min(i + 3, len(lines)))
                if j == i or "|" in lines[j]}
        lines = [l for i, l in enumerate(lines) if i not in drop]
    out = "\n".join(l for l in lines
                    if "packed-fp32-ops" not in l and l.strip() != "1 warning generated.")
    if r.returncode != 0:
        raise RuntimeError("build failed: " + " ".join(cmd) + "\n" + r.stdout)
    if out.strip():
        sys.stderr.write(out + "\n")


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    objs = []
    for src in ("analyze.cpp",):
        obj = os.path.join(BUILD, src + ".o")
        _run([HIPCC, *COMMON, "-c", os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    for src in KERNEL_FILES:
        obj = os.path.join(BUILD, src + ".o")
        _run([HIPCC, *COMMON, *DEVICE_FLAGS, *FILE_OPT.get(src, []), USAGE, "-c",
              os.path.join(CSRC, src), "-o", obj])
        objs.append(obj)
    tmp = LIB + ".tmp"
    _run([HIPCC, "-shared", "-fPIC", *DEVICE_FLAGS, "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
