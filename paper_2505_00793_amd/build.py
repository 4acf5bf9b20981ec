"""Build libmfmg.so (HIP, gfx950) in-tree with hipcc.

    python -m paper_2505_00793_amd.build                 # rebuild everything
    python -m paper_2505_00793_amd.build api.hip ...     # recompile these, relink
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD_DIR = os.path.join(ROOT, "_build")
LIB = os.path.join(HERE, "libmfmg.so")
GEMM_PARTS = 9   # gemm.hip is compiled in parts (its kernel instances), side by side
SOURCES = ["gemm.hip", "elementwise.hip", "linreg.hip", "transformer.hip", "attention.hip", "tf_engine.hip", "api.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    f"-I{os.path.join(ROOT, 'include')}",
    # no packed-fp32 instructions in device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _units(src: str):
    """(object, extra flags) of each translation unit of a source."""
    stem = os.path.join(BUILD_DIR, os.path.splitext(src)[0])
    if src == "gemm.hip":
        return [(f"{stem}_{k}.o", [f"-DGEMM_PART={k}"]) for k in range(GEMM_PARTS)]
    return [(stem + ".o", [])]


def _compile(job) -> None:
    src, obj, extra = job
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")


def build(verbose: bool = True, only=None) -> str:
    """Compile every source (or only the named ones, reusing the other objects)
    and link the shared library; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    todo = SOURCES if not only else [s for s in SOURCES if s in only]
    if only and len(todo) != len(set(only)):
        raise ValueError(f"unknown sources in {only}; sources are {SOURCES}")
    jobs = [(s, obj, extra) for s in todo for obj, extra in _units(s)]
    with cf.ThreadPoolExecutor(max_workers=8) as ex:
        list(ex.map(_compile, jobs))
    objs = [obj for s in SOURCES for obj, _ in _units(s)]
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-o", tmp, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    os.replace(tmp, LIB)
    if verbose:
        print(f"built {LIB}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build(only=sys.argv[1:] or None)
