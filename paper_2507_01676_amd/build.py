"""Builds libembx.so (HIP kernels for gfx950 + the C ABI + the host planner) in-tree.

    python paper_2507_01676_amd/build.py
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libembx.so")
# the same library, except that the 12-load gather kernels rebase their positions after at most
# FAR lookups instead of 2^30, so that tests reach that code with ordinary batches
FAR_LIB = os.path.join(HERE, "libembx_far.so")
FAR = 100
ARCH = "gfx950"

HIP_FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-ffp-contract=off",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
             "-I", os.path.join(ROOT, "include")]
# For kernels whose control flow is wave-uniform: leave it as written instead of turning every branch
# into the flag-guarded form that divergent branches need (a compare, a jump and the additions per
# instruction of a step, against about twenty instructions)
UNIFORM_FLAGS = ["-mllvm", "-structurizecfg-skip-uniform-regions=1"]
HOST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math", "-Wall"]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"build step failed: {' '.join(cmd[:3])} ...")
    return r


# lookup.hip is compiled in parts (EMBX_PART): one per (row type, weighted) kernel family of
# staged plans and of gather-only ones, plus the probes, filler and launch code, plus one per
# family of gather-only kernels with wave-uniform control
LOOKUP_PARTS = 12
LOOKUP_UNIFORM_PARTS = (5, 6, 11)
# gather.hip: one part per (row type, weighted) kernel family, each built for every number
# of row loads in flight per step a plan may choose (kGatherStepChoices in device_types.hpp)
GATHER_PARTS = 4
GATHER_STEPS = (12, 13, 16)


def _run_all(cmds, verbose):
    """Runs the compile commands in parallel; raises on the first failure."""
    procs = []
    for cmd in cmds:
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    failed = None
    for cmd, p in procs:
        out, _ = p.communicate()
        if p.returncode != 0 and failed is None:
            failed = (cmd, out)
    if failed is not None:
        sys.stderr.write(failed[1])
        raise RuntimeError(f"build step failed: {' '.join(failed[0][:3])} ...")


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD, exist_ok=True)
    hipcc = _hipcc()
    cmds, objs = [], []
    for part in range(LOOKUP_PARTS):
        o = os.path.join(BUILD, f"lookup_{part}.o")
        uniform = UNIFORM_FLAGS if part in LOOKUP_UNIFORM_PARTS else []
        cmds.append([hipcc, *HIP_FLAGS, *uniform, f"-DEMBX_PART={part}", "-c", os.path.join(CSRC, "lookup.hip"), "-o", o])
        objs.append(o)
    for ks in GATHER_STEPS:
        for part in range(GATHER_PARTS):
            o = os.path.join(BUILD, f"gather_{part}_k{ks}.o")
            cmds.append([hipcc, *HIP_FLAGS, *UNIFORM_FLAGS, f"-DEMBX_GPART={part}", f"-DEMBX_GKS={ks}", "-c",
                         os.path.join(CSRC, "gather.hip"), "-o", o])
            objs.append(o)
    far = {}
    for part in range(GATHER_PARTS):
        o = os.path.join(BUILD, f"gather_{part}_k12_far.o")
        cmds.append([hipcc, *HIP_FLAGS, *UNIFORM_FLAGS, f"-DEMBX_GPART={part}", "-DEMBX_GKS=12", f"-DEMBX_FAR={FAR}",
                     "-c", os.path.join(CSRC, "gather.hip"), "-o", o])
        far[os.path.join(BUILD, f"gather_{part}_k12.o")] = o
    o = os.path.join(BUILD, "api.o")
    cmds.append([hipcc, *HIP_FLAGS, "-x", "hip", "-c", os.path.join(CSRC, "api.cpp"), "-o", o])
    objs.append(o)
    # the planner is plain host C++: every binary64 operation rounds as written
    for name in ("planner", "queues"):
        o = os.path.join(BUILD, f"{name}.o")
        cmds.append(["g++", *HOST_FLAGS, "-c", os.path.join(CSRC, f"{name}.cpp"), "-o", o])
        objs.append(o)
    _run_all(cmds, verbose)
    for lib, parts in ((FAR_LIB, [far.get(o, o) for o in objs]), (LIB, objs)):
        tmp = lib + ".tmp"
        _run([hipcc, "-shared", f"--offload-arch={ARCH}", "-o", tmp, *parts], verbose)
        os.replace(tmp, lib)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
