"""Compile libgpuqt.so for gfx950 in-tree with hipcc (used by __graft_entry__.build)."""
from __future__ import annotations

import concurrent.futures
import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libgpuqt.so")
BUILD_DIR = os.path.join(ROOT, "_build")

SOURCES = ["kernels.hip", "kernels_kpm.hip", "kernels_adjoint.hip", "kernels_adjoint_pair.hip", "kernels_adjoint_sym.hip", "api.cpp", "layout.cpp", "io.cpp", "tune.cpp", "noalloc.hip",
           "lattice.cpp", "march.hip", "march_square_uniform.hip", "march_square_real.hip", "march_square_complex.hip", "march_square_dict.hip",
           "march_brick_uniform.hip", "march_brick_real.hip", "march_brick_complex.hip", "march_brick_dict.hip",
           "march_box_uniform.hip",
           "patch_square_uniform.hip", "patch_square_real.hip", "patch_square_complex.hip", "patch_square_dict.hip",
           "patch_brick_uniform.hip", "patch_brick_real.hip", "patch_brick_complex.hip", "patch_brick_dict.hip",
           "patch_chain.hip",
           "patch_nnn_uniform.hip", "patch_nnn_real.hip", "patch_nnn_complex.hip", "patch_nnn_dict.hip"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include")]


def _hipcc() -> str:
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found")
    return p


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    lines = [ln for ln in r.stdout.splitlines() if "packed-fp32-ops" not in ln]
    if r.returncode != 0:
        raise RuntimeError("build failed:\n" + " ".join(cmd) + "\n" + "\n".join(lines))
    return lines


def build(verbose: bool = False) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    hipcc = _hipcc()
    objs = []
    cmds = []
    for src in SOURCES:
        obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
        objs.append(obj)
        cmds.append([hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj])
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(len(cmds), os.cpu_count() or 8)) as ex:
        for lines in ex.map(_run, cmds):
            if verbose:
                print("\n".join(lines))
    tmp = OUT + ".tmp"
    _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
