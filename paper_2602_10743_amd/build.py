"""Build the KLA HIP library for gfx950, paper_2602_10743_amd/libkla.so, and the native part
of its Python binding, _kla_torch.so (plain C++ against torch's headers).

Every HIP source is compiled with hipcc for gfx950 only, with packed-fp32
instruction selection disabled, and linked with the C ABI into one shared
library that exports the functions declared in include/kla.h.
"""
import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libkla.so")
EXT = os.path.join(HERE, "_kla_torch.so")
BUILD_DIR = os.path.join(HERE, "_build")

ARCH = "gfx950"
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=fast", "-munsafe-fp-atomics",
    "-I", INCLUDE, "-I", CSRC, "-Wall", "-Wno-unused-function",
]
SOURCES = ["kla_api.cpp", "recurrent.hip", "validate.hip", "ou.hip", "pc.hip", "block.hip", "chunk_fwd.hip",
           "chunk_seg.hip", "chunk_bwd_dv.hip", "chunk_bwd_dk.hip", "chunk64.hip", "chunk64_par.hip",
           "noalloc.hip", "mc.hip"]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the KLA library needs ROCm's hipcc to build")


def _binding_flags():
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    rocm = os.path.dirname(os.path.dirname(_hipcc()))
    inc = include_paths() + [sysconfig.get_paths()["include"], os.path.join(rocm, "include"), INCLUDE]
    compile_ = ["-O2", "-std=c++17", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + [f"-I{p}" for p in inc]
    link = [f"-L{p}" for p in library_paths()] + ["-lc10", "-lc10_hip", "-ltorch", "-ltorch_cpu", "-ltorch_python",
                                                  f"-L{HERE}", "-l:libkla.so", "-Wl,-rpath,$ORIGIN"]
    return compile_, link


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(BUILD_DIR, exist_ok=True)
    hipcc = _hipcc()
    cxx = os.environ.get("CXX") or shutil.which("g++") or "c++"
    cxxflags, ldflags = _binding_flags()
    binding = os.path.join(BUILD_DIR, "binding.o")

    def compile_binding():
        subprocess.run([cxx, *cxxflags, "-c", os.path.join(CSRC, "binding.cpp"), "-o", binding], check=True)

    def compile_one(src):
        obj = os.path.join(BUILD_DIR, os.path.splitext(src)[0] + ".o")
        lang = ["-x", "hip"]
        cmd = [hipcc, *lang, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        native = ex.submit(compile_binding)
        objs = list(ex.map(compile_one, SOURCES))
        native.result()
    tmp = LIB + ".tmp"
    cmd = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    subprocess.run([cxx, "-shared", binding, "-o", EXT + ".tmp", *ldflags], check=True)
    os.replace(EXT + ".tmp", EXT)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
