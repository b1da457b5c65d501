"""Builds libnats.so (HIP kernels + C ABI) for gfx950 with hipcc, and the host extension _nats_host, in-tree."""
from __future__ import annotations

import os
import subprocess
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libnats.so")
HOST = os.path.join(PKG, "_nats_host" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
         # keep the compiler from forming packed-fp32 VALU ops
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def sources():
    return sorted(f for f in os.listdir(CSRC) if f.endswith(".hip"))


def compile_host() -> str:
    """csrc/host.cpp, plain C++ against torch's headers."""
    import torch
    from torch.utils import cpp_extension
    obj = os.path.join(OBJ, "host.o")
    inc = cpp_extension.include_paths() + ["/opt/rocm/include", sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    # NDEBUG: pybind11's debug counters, which come in with torch's headers, are thread-local variables.  A library with those that
    # is loaded last and never touches them makes every thread-local access of the process take glibc's slow path (2.35; torch
    # makes several per call: torch.empty 1.5 -> 1.8 us, a prefill's host side 35 -> 39).
    cmd = (["g++", "-O2", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-w", "-DNDEBUG", "-DUSE_ROCM", "-D__HIP_PLATFORM_AMD__=1",
            f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"] + ["-I" + i for i in inc]
           + ["-c", os.path.join(CSRC, "host.cpp"), "-o", obj])
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed for host.cpp:\n{r.stderr}")
    return obj


def link_host(obj: str) -> None:
    import torch
    tlib = os.path.join(os.path.dirname(torch.__file__), "lib")
    r = subprocess.run(["g++", "-shared", "-o", HOST, obj, "-L" + PKG, "-l:libnats.so", "-Wl,-rpath,$ORIGIN", "-L" + tlib,
                        "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")


def build_library(verbose: bool = False) -> str:
    """Compile every csrc/*.hip and link libnats.so.  Always recompiles."""
    os.makedirs(OBJ, exist_ok=True)

    def compile_one(src):
        obj = os.path.join(OBJ, src[:-4] + ".o")
        cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed for {src}:\n{r.stderr}")
        if verbose:
            print("compiled", src)
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(sources()))) as ex:
        host = ex.submit(compile_host)   # the longest of them: torch's headers
        objs = list(ex.map(compile_one, sources()))
        host_obj = host.result()
    r = subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs,
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    link_host(host_obj)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
