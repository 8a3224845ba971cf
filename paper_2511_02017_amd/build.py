"""Builds libtapout.so (HIP, gfx950) in-tree with hipcc, and _marshal.so, the binding's native part, with g++.

Run as `python -m paper_2511_02017_amd.build`.  hipcc cross-compiles without a
GPU, so this works on a CPU-only machine.  With `--stamps` it builds
libtapout_stamps.so beside it instead: the same sources with per-workgroup time
stamps in the final-token kernels (see wg_stamps.py), for measurements only.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(PKG, "libtapout.so")
MARSHAL = os.path.join(PKG, "_marshal.so")
LIB_STAMPS = os.path.join(PKG, "libtapout_stamps.so")
SOURCES = ["row_reduce.hip", "finalize.hip", "verify.hip", "bandit.hip", "api.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden",
    "-ffp-contract=off",                     # every fused multiply-add in the sources is written explicitly
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def build(verbose: bool = False, extra_flags=(), stamps: bool = False) -> str:
    obj_dir = os.path.join(OBJ, "stamps") if stamps else OBJ
    lib = LIB_STAMPS if stamps else LIB
    if stamps:
        extra_flags = (*extra_flags, "-DTAPOUT_WG_STAMPS")
    os.makedirs(obj_dir, exist_ok=True)
    cc = hipcc()

    def compile_one(src):
        obj = os.path.join(obj_dir, src.replace(".hip", ".o"))
        cmd = [cc, *FLAGS, *extra_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
        warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if verbose and warn:
            print(warn, flush=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    cmd = [cc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", lib]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    return lib


def build_marshal() -> str:
    """_marshal.so, the native argument marshalling of binding.py: host code against torch's own headers and libraries."""
    import sysconfig

    from torch.utils import cpp_extension
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc()))) if os.path.sep in hipcc() else "/opt/rocm"
    if not os.path.isdir(os.path.join(rocm, "include", "hip")):
        rocm = "/opt/rocm"
    libs = cpp_extension.library_paths()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
           "-D_GLIBCXX_USE_CXX11_ABI=" + ("1" if __import__("torch")._C._GLIBCXX_USE_CXX11_ABI else "0"),
           "-I", os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"], "-isystem", os.path.join(rocm, "include"),
           *(a for p in cpp_extension.include_paths() for a in ("-isystem", p)), os.path.join(CSRC, "marshal.cpp"),
           *(a for p in libs for a in ("-L", p)), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-ldl", "-o", MARSHAL]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on marshal.cpp:\n{r.stdout}\n{r.stderr}")
    return MARSHAL


if __name__ == "__main__":
    print(build_marshal())
    print(build(verbose="-v" in sys.argv, stamps="--stamps" in sys.argv))
