"""Builds libnm_sparse.so (HIP, gfx950 only) in-tree with hipcc, and the native marshalling of the calls of a layer."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

from .binding import calls_path

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libnm_sparse.so")
SOURCES = ("nm_api.hip", "nm_direct.hip", "nm_fewtok.hip", "nm_grad.hip", "nm_int8.hip", "nm_pack.hip", "nm_probe.hip", "nm_rank.hip", "nm_search.hip", "nm_spmm.hip")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++20", "-fPIC", "-fno-gpu-rdc",
    # packed fp32 ALU forms are switched off for this target
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument", "-Wno-inline-asm",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: the HIP library cannot be built")
    return exe


def compile_calls(source: str, path: str) -> None:
    """Compile the host-only extension that reads torch tensors (against the installed torch)."""
    from torch.utils import cpp_extension
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    includes = [os.path.join(ROOT, "include"), *cpp_extension.include_paths(), os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    tmp = path + ".tmp"
    cmd = ["g++", "-O2", "-std=c++20", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           *[f"-I{p}" for p in includes], source, "-o", tmp,
           *[f"-L{p}" for p in cpp_extension.library_paths()], "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-lc10_hip"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"compiling {source} failed:\n{res.stderr}")
    os.replace(tmp, path)


def build_library(verbose: bool = False) -> str:
    """Compile every translation unit and link the shared library, and the extension beside it; returns the library's path.
    The library knows nothing of torch: it is in place also where the extension, reported last, could not be built."""
    obj_dir = os.path.join(PKG_DIR, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    cc = hipcc()

    def compile_one(src: str) -> str:
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [cc, *HIPCC_FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l)
        if res.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=len(SOURCES) + 1) as pool:
        calls = pool.submit(lambda: compile_calls(os.path.join(CSRC, "nm_calls.cpp"), calls_path()))
        objs = list(pool.map(compile_one, SOURCES))
    tmp = LIB_PATH + ".tmp"
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", "-fno-gpu-rdc", *objs, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"link failed:\n{res.stderr}")
    os.replace(tmp, LIB_PATH)
    calls.result()
    return LIB_PATH


if __name__ == "__main__":
    print(build_library(verbose=True))
