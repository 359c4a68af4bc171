"""Compile libpab.so (HIP, gfx950 only) in-tree with hipcc, and the CPython binding of its two hottest calls with g++.

The library needs hipcc and nothing else.  The binding is for Python callers, who do without it where it cannot be built."""
from __future__ import annotations

import importlib.metadata
import os
import re
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libpab.so")
SOURCES = [os.path.join(CSRC, "pab_api.hip")]
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # packed fp32 VALU forms stay off for device code (the host pass does not know the
    # feature and says so; that warning is harmless)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # MFMA results feed VALU code (softmax): select the VGPR form so that no accumulator has to be
    # copied between the AGPR and VGPR halves of the register file
    "-mllvm", "-amdgpu-mfma-vgpr-form",
    # no NaN bookkeeping in max chains (masked scores are -inf, never NaN)
    "-fno-honor-nans",
    "-Wno-unused-command-line-argument",
]


def build_lib(verbose: bool = False, extra_flags=()) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + ["-o", tmp] + SOURCES
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        sys.stderr.write(out + "\n")
        raise RuntimeError("hipcc failed building libpab.so")
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB)
    return LIB


def binding_path(torch_version: str | None = None) -> str:
    """Where the binding for this Python and this torch (the installed one unless given) lies: it fits no other of either."""
    version = re.sub(r"[^0-9a-zA-Z]+", "_", torch_version or importlib.metadata.version("torch"))
    return os.path.join(HERE, "_binding_torch_%s%s" % (version, sysconfig.get_config_var("EXT_SUFFIX")))


def build_binding(verbose: bool = False) -> str:
    """The CPython binding (csrc/pab_binding.cpp), against the installed torch and the libpab.so beside it."""
    import torch
    root = os.path.dirname(torch.__file__)
    path = binding_path(torch.__version__)
    tmp = path + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I" + os.path.join(root, "include"),
           "-I" + os.path.join(root, "include", "torch", "csrc", "api", "include"), "-I" + sysconfig.get_paths()["include"],
           os.path.join(CSRC, "pab_binding.cpp"), "-o", tmp, "-L" + HERE, "-l:" + os.path.basename(LIB),
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-Wl,-rpath,$ORIGIN"]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + "\n")
        raise RuntimeError("%s failed building %s" % (cmd[0], os.path.basename(path)))
    os.replace(tmp, path)
    return path


def build_binding_if_possible(verbose: bool = False) -> str | None:
    """build_binding, or None and the reason on stderr where there is no torch or no compiler for it."""
    try:
        return build_binding(verbose)
    except (ImportError, OSError, RuntimeError) as e:
        sys.stderr.write("the native binding is not built (%s): calls from Python go through ctypes\n" % e)
        return None


def ensure_built() -> str:
    """Build only what is not there: callers load what is built."""
    if not os.path.exists(LIB):
        build_lib()
    try:
        missing = not os.path.exists(binding_path())
    except importlib.metadata.PackageNotFoundError:   # no torch: none to bind
        missing = False
    if missing:
        build_binding_if_possible()
    return LIB


def device_asm(path: str, extra_flags=()) -> str:
    """Write the gfx950 assembly of the device code (same flags as the library) to `path`."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    cmd = [hipcc] + flags + list(extra_flags) + ["-S", "--cuda-device-only", "-o", path] + SOURCES
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        sys.stderr.write(res.stdout + "\n")
        raise RuntimeError("hipcc failed writing the device assembly")
    return path


if __name__ == "__main__":
    print(build_lib(verbose=True))
    print(build_binding_if_possible(verbose=True))
