"""Builds libmhcl.so (HIP, gfx950 only) next to this file with hipcc, the graph nodes of autograd.py
(torch_ext/autograd.cpp -> _autograd_native.so), and the stand-alone
memory-system probe (probe/memsys_probe.hip -> memsys_probe) that `bench.py --memsys` runs."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libmhcl.so")
OBJ_DIR = os.path.join(_HERE, "_build")
PROBE_SRC = os.path.join(_HERE, "probe", "memsys_probe.hip")
PROBE = os.path.join(_HERE, "memsys_probe")

AUTOGRAD_SRC = os.path.join(_HERE, "torch_ext", "autograd.cpp")
AUTOGRAD = os.path.join(_HERE, "_autograd_native.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
    # hipcc -O3 may otherwise fuse scalar fp32 code into packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".hip"))


def build_library(verbose: bool = False) -> str:
    os.makedirs(OBJ_DIR, exist_ok=True)
    srcs = sources()
    objs = [os.path.join(OBJ_DIR, os.path.basename(s) + ".o") for s in srcs]

    def compile_one(pair):
        src, obj = pair
        cmd = [HIPCC, *FLAGS, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        return src, r

    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        for src, r in ex.map(compile_one, zip(srcs, objs)):
            # the host pass warns that it does not know the packed-fp32 feature: harmless
            err = "\n".join(l for l in r.stderr.splitlines()
                            if "packed-fp32-ops" not in l and l.strip())
            if r.returncode != 0:
                raise RuntimeError(f"hipcc failed on {src}:\n{r.stderr}")
            if err and verbose:
                print(err, file=sys.stderr)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stderr}")
    build_autograd(verbose)
    build_probe(verbose)
    return LIB


def build_autograd(verbose: bool = False) -> str:
    """The graph nodes of autograd.py as a Python extension (host code; linked with libmhcl.so and torch)."""
    from torch.utils.cpp_extension import include_paths
    import torch
    lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    name = os.path.basename(AUTOGRAD).split(".")[0]
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", f"-DTORCH_EXTENSION_NAME={name}",
           "-DTORCH_API_INCLUDE_EXTENSION_H", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-I{p}" for p in include_paths()], "-I/opt/rocm/include",
           f"-I{sysconfig.get_paths()['include']}", AUTOGRAD_SRC, "-o", AUTOGRAD, f"-L{lib}", "-ltorch_python", "-ltorch",
           "-ltorch_cpu", "-lc10", "-lc10_hip", f"-L{_HERE}", "-lmhcl", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"g++ failed on {AUTOGRAD_SRC}:\n{r.stderr}")
    return AUTOGRAD


def build_probe(verbose: bool = False) -> str:
    """The traffic-skeleton executable (no part of the library; it links nothing of it)."""
    cmd = [HIPCC, *[f for f in FLAGS if f != "-fPIC"], PROBE_SRC, "-o", PROBE]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {PROBE_SRC}:\n{r.stderr}")
    return PROBE


if __name__ == "__main__":
    print(build_library(verbose=True))
