"""Build the C-ABI library ``libcg_conv.so`` from ``csrc/`` with hipcc for gfx950, and the binding's ``_calls.so`` (host code) with g++."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor
from pathlib import Path

PKG = Path(__file__).resolve().parent
ROOT = PKG.parent
CSRC = PKG / "csrc"
LIB = PKG / "libcg_conv.so"
CALLS = PKG / "_calls.so"

SOURCES = ["cg_conv_api.hip", "kernels_naive.hip", "kernels_direct.hip", "kernels_rows.hip", "kernels_counts.hip", "kernels_dense.hip",
           "kernels_tile.hip", "kernels_tile_bf16_k3.hip", "kernels_tile_bf16_k1.hip", "kernels_tile_i8_k3.hip",
           "kernels_tile_i8_k1.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # accumulators stay in ordinary vector registers: with the AGPR form the compiler copies them
    # back and forth around the branches inside the MFMA loops and mis-counts the wait states
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-warning-option",
]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


def calls_command(out, lib_dir) -> list:
    """g++ on the Python extension of the calls (csrc/py_calls.cpp), against torch's C++ interface and the library in lib_dir."""
    import torch
    home = Path(torch.__file__).resolve().parent
    rocm = Path(hipcc()).resolve().parent.parent
    rocm = rocm if (rocm / "include" / "hip").is_dir() else Path("/opt/rocm")
    return ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
            "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DCG_TORCH_VERSION="%s"' % torch.__version__, "-isystem", str(home / "include"),
            "-isystem", str(home / "include" / "torch" / "csrc" / "api" / "include"), "-isystem", str(rocm / "include"),
            "-isystem", sysconfig.get_paths()["include"], "-I", str(ROOT / "include"), "-I", str(CSRC), str(CSRC / "py_calls.cpp"), "-o", str(out),
            "-L", str(home / "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python", "-L", str(lib_dir), "-lcg_conv", "-Wl,-rpath,$ORIGIN"]


def build(verbose: bool = False, extra=(), jobs: int = 6) -> Path:
    """Compile every source every time it is called (the 'does it build' check): one object per
    source, compiled side by side, then the two links."""
    cc = hipcc()
    work = Path(tempfile.mkdtemp(prefix="cg_build_"))
    try:
        def compile_one(src: str) -> str:
            obj = work / (src + ".o")
            cmd = [cc, *FLAGS, *extra, "-I", str(ROOT / "include"), "-I", str(CSRC), "-c", str(CSRC / src),
                   "-o", str(obj)]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return str(obj)

        with ThreadPoolExecutor(max_workers=max(1, jobs)) as pool:
            objs = list(pool.map(compile_one, SOURCES))
        # both are linked before either is put in place: a library beside an extension of another build would be called with other arguments
        lib, calls = work / LIB.name, work / CALLS.name
        for link in ([cc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", str(lib)], calls_command(calls, work)):
            if verbose:
                print(" ".join(link), flush=True)
            subprocess.check_call(link)
        placed = [(to.with_name(to.name + ".tmp%d" % os.getpid()), to) for to in (LIB, CALLS)]
        for built, (tmp, _) in zip((lib, calls), placed):
            shutil.copy(built, tmp)
        for tmp, to in placed:
            os.replace(tmp, to)
    finally:
        shutil.rmtree(work, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
