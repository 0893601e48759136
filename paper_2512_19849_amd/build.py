"""Builds libep.so (HIP kernels + host proxy) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import shutil
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libep.so")
CALL = os.path.join(HERE, "_epcall.so")
CALL_SRC = os.path.join(CSRC, "pycall.cpp")
SOURCES = ["layout.hip", "dispatch.hip", "combine.hip", "ht_ring.hip", "service.hip", "proxy.cpp", "api.cpp"]
HEADERS = ["ep_internal.h", "ep_device.h", "ep_host.h", os.path.join("..", "..", "include", "ep.h"),
           os.path.join("..", "..", "include", "ep_diag.h")]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", shutil.which("hipcc")):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


def _torch_version() -> str:
    """The version of the torch that runs, empty where there is none: libep.so needs none."""
    try:
        import torch
    except ImportError:
        return ""
    return torch.__version__


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + HEADERS)


def call_stale() -> bool:
    """_epcall is missing, older than what it is built from, or built for another torch (it carries the version's text)."""
    if not os.path.exists(CALL):
        return True
    t = os.path.getmtime(CALL)
    if any(os.path.getmtime(f) > t for f in (CALL_SRC, os.path.join(HERE, "..", "include", "ep.h"))):
        return True
    version = _torch_version()
    with open(CALL, "rb") as f:
        return bool(version) and f"torch {version}\0".encode() not in f.read()


def build_lib(force: bool = True, verbose: bool = False) -> str:
    """Compile every HIP/C++ source of the library for gfx950 into libep.so, and the module that calls it from Python.
    The library needs neither torch nor g++; without them it is built alone, and the binding calls it through ctypes."""
    if force or stale():
        objs = []
        common = ["-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function"]
        for src in SOURCES:
            obj = os.path.join(CSRC, src + ".o")
            cmd = [hipcc(), *common, "-c", os.path.join(CSRC, src), "-o", obj]
            if src.endswith(".hip"):
                # packed fp32 ALU forms are kept off for all device code
                cmd[1:1] = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
            if verbose:
                print(" ".join(cmd))
            subprocess.run(cmd, check=True)
            objs.append(obj)
        cmd = [hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs, "-lpthread"]
        if verbose:
            print(" ".join(cmd))
        subprocess.run(cmd, check=True)
    if force or call_stale():
        build_call(verbose)
    return LIB


def build_call(verbose: bool = False) -> None:
    """_epcall, the module that takes tensors to the calls of a step (host code only)."""
    import sysconfig

    if os.path.exists(CALL):
        os.remove(CALL)  # (what is out of date is not left behind, whether or not a new one can be made)
    if not _torch_version() or not shutil.which("g++"):
        print(f"{os.path.basename(CALL)} is not built (it needs torch and g++): calls go through ctypes")
        return
    import torch
    home = os.path.dirname(torch.__file__)
    lib = os.path.join(home, "lib")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f'-DEP_TORCH="{_torch_version()}"',
           "-I" + os.path.join(home, "include"), "-I" + os.path.join(home, "include", "torch", "csrc", "api", "include"),
           "-I" + sysconfig.get_paths()["include"], "-I/opt/rocm/include", CALL_SRC, "-o", CALL, "-L" + HERE, "-l:libep.so",
           "-L" + lib, "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10", "-lc10_hip", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)


PROBE_SRC = os.path.join(HERE, "probes", "mem_patterns.hip")
PROBE_BIN = os.path.join(HERE, "probes", "mem_patterns")


def build_probes(verbose: bool = False) -> str:
    """The stand-alone access-pattern probe (a measuring program for rocprofv3, not part of the library)."""
    cmd = [hipcc(), "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", PROBE_SRC, "-o", PROBE_BIN]
    if verbose:
        print(" ".join(cmd))
    subprocess.run(cmd, check=True)
    return PROBE_BIN


if __name__ == "__main__":
    print(build_lib(verbose=True))
    print(build_probes(verbose=True))
