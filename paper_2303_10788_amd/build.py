"""Build libccut.so for gfx950 with hipcc (in-tree, no JIT cache).

    python -m paper_2303_10788_amd.build
"""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG, "csrc")
OUT = os.path.join(PKG, "libccut.so")
PACK_OUT = os.path.join(PKG, "libccut_pack" + sysconfig.get_config_var("EXT_SUFFIX"))
BUILD_DIR = os.path.join(PKG, "_build")
SOURCES = ["plan.cpp", "cutfind.cpp", "api.cpp", "k_sample.hip", "k_sv.hip", "k_contract.hip", "k_heis.hip",
           "k_exact.hip", "k_gemm.hip", "k_mlp.hip", "k_train.hip", "k_mlc.hip", "k_affine.hip"]
ARCH = os.environ.get("CCUT_OFFLOAD_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _flags():
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-I", os.path.join(PKG, "..", "include")]


def _compile(src: str) -> str:
    obj = os.path.join(BUILD_DIR, os.path.basename(src) + ".o")
    cmd = [hipcc(), *_flags(), "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"compile failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    return obj


def _build_pack() -> None:
    """The binding's conversion of Python circuits (its symbols of the
    interpreter resolve in the process that loads it).  Built against one
    interpreter, whose tag is in its name; the binding does without it, so a
    build that lacks the interpreter's headers only says so."""
    tmp = PACK_OUT + f".tmp{os.getpid()}"
    cmd = [hipcc(), "-no-hip-rt", "-x", "c++", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-I", os.path.join(PKG, "..", "include"), "-I", sysconfig.get_paths()["include"],
           os.path.join(CSRC, "pack.cpp"), "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode == 0:
        os.replace(tmp, PACK_OUT)
        return
    if os.path.exists(PACK_OUT):
        os.remove(PACK_OUT)
    print(f"the native conversion of circuits is left out: {' '.join(cmd)}\n{r.stderr}", file=sys.stderr, flush=True)


def build(verbose: bool = False, jobs: int = 8) -> str:
    """Compile every source and link libccut.so; returns its path."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    with cf.ThreadPoolExecutor(max_workers=jobs) as ex:
        pack = ex.submit(_build_pack)
        objs = list(ex.map(_compile, SOURCES))
        pack.result()
    tmp = OUT + f".tmp{os.getpid()}"
    # -z defs: an unresolved symbol fails the link instead of the first load
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-shared", "-fPIC", "-Wl,-z,defs", *objs, "-o", tmp]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed: {' '.join(cmd)}\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, OUT)
    if verbose:
        print("built", OUT)
    return OUT


if __name__ == "__main__":
    build(verbose=True)
    sys.exit(0)
