"""Build libpe.so (the C-ABI library of HIP kernels) for gfx950 with hipcc, and behind it _pe_host.so (native argument marshalling of
its Python front end) with g++ where there is torch, in-tree."""
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpe.so")
HOST_LIB = os.path.join(HERE, "_pe_host.so")
SOURCES = ["pe_api.hip", "score_blocks.hip", "evict_blocks.hip", "paged_decode.hip", "paged_decode_bf16.hip",
           "prefill_prune.hip"]
# Packed fp32 VALU ops are switched off for all device code.  The leading kernel arguments (up to 14 dwords) are preloaded
# into scalar registers instead of being loaded by every wave.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-kernarg-preload-count=14"]


def build(verbose: bool = False, extra_flags=()) -> str:
    os.makedirs(BUILD, exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    procs = []
    for src in SOURCES:
        obj = os.path.join(BUILD, src.replace(".hip", ".o"))
        cmd = [hipcc] + FLAGS + list(extra_flags) + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, obj, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    objs, failed = [], []
    for src, obj, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l and l.strip())
        if p.returncode != 0:
            failed.append((src, out))
        elif out and verbose:
            print(out)
        objs.append(obj)
    if failed:
        raise RuntimeError("hipcc failed:\n" + "\n".join("%s:\n%s" % f for f in failed))
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, check=True)
    os.replace(tmp, LIB)
    build_c_smoke()
    build_host(verbose)
    return LIB


def build_host(verbose: bool = False):
    """Compile the Python extension (host code only).  The C library is there without it, and needs neither Python nor torch: without
    torch there is no Python front end to build it for."""
    import importlib.util
    import sysconfig
    if importlib.util.find_spec("torch") is None:
        return None
    import torch
    from torch.utils import cpp_extension
    tmp = HOST_LIB + ".tmp.%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unused-function", "-Wno-attributes",
           "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + sysconfig.get_paths()["include"]]
    cmd += ["-isystem" + d for d in cpp_extension.include_paths("cuda")]
    cmd += [os.path.join(CSRC, "pe_host.cpp"), "-o", tmp] + ["-L" + d for d in cpp_extension.library_paths("cuda")]
    cmd += ["-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if p.returncode != 0:
        raise RuntimeError("g++ failed on pe_host.cpp (libpe.so is built):\n" + p.stdout)
    os.replace(tmp, HOST_LIB)
    return HOST_LIB


C_SMOKE_SRC = os.path.join(os.path.dirname(HERE), "tests", "c_abi", "pe_c_smoke.c")
C_SMOKE_BIN = os.path.join(HERE, "pe_c_smoke")


def build_c_smoke() -> str:
    """A plain-C program that drives libpe through the C ABI (used by a GPU test); built with gcc."""
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    cmd = ["gcc", "-std=c11", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-o",
           C_SMOKE_BIN, C_SMOKE_SRC, "-L", HERE, "-lpe", "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-lm",
           "-Wl,-rpath,$ORIGIN", "-Wl,-rpath," + os.path.join(rocm, "lib")]
    subprocess.run(cmd, check=True)
    return C_SMOKE_BIN


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
