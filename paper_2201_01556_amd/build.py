"""Build ``libhyperflow.so`` (HIP, gfx950) in-tree with hipcc.

Usage: ``python -m paper_2201_01556_amd.build`` (or ``build_library()``).
Objects go to ``_build/`` at the repository root; the shared library lands
next to this file.
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(ROOT, "_build")
LIB = os.path.join(PKG, "libhyperflow.so")

SOURCES = ["hf_build.hip", "hf_solve.hip", "hf_batch.hip", "hf_mlp.hip", "hf_api.hip",
           "hf_noalloc.hip", "hf_regions.hip", "hf_moves.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-fvisibility=hidden",
    # packed fp32 VALU ops stay disabled (no such code is wanted here)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
    "-I" + INCLUDE,
    "-I" + CSRC,
]


# registers, spills and LDS of every kernel, read by register_spills
REMARKS = "-Rpass-analysis=kernel-resource-usage"


def register_spills(remarks: str) -> dict:
    """Vector registers that each of the library's own kernels spills, from
    the compiler's resource remarks (kernels of library headers left out)."""
    out, name = {}, None
    for line in remarks.splitlines():
        if "Function Name:" in line:
            name = line.split("Function Name:")[1].split()[0]
        elif "VGPRs Spill:" in line and name and name.startswith("_ZN2hf"):
            out[name] = int(line.split("VGPRs Spill:")[1].split()[0])
    return out


def compile_source(src: str, obj: str) -> None:
    """Compile one source file.  A kernel that spills vector registers is
    refused: a form of k_batch_wg with spills once left the source sides
    unwritten while its flows were right, for a cause that was not found."""
    r = subprocess.run([HIPCC, *FLAGS, REMARKS, "-c", src, "-o", obj], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed for {src}:\n{r.stdout}\n{r.stderr}")
    spills = {k: n for k, n in register_spills(r.stderr).items() if n}
    if spills:
        os.remove(obj)
        raise RuntimeError(f"{src}: kernels spill vector registers: {spills}")


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    compile_source(os.path.join(CSRC, src), obj)
    return obj


def build_library(verbose: bool = False) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
    sys.exit(0)
