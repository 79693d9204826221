"""Builds libactq.so in-tree with hipcc for gfx950 (cross-compiles without a GPU), and actq_torch.so, the
binding's native half, with the host compiler against torch's headers."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
CSRC = os.path.join(_HERE, "csrc")
LIB = os.path.join(_HERE, "libactq.so")
SOURCES = ["actq_api.cpp", "actq_kernels.hip", "actq_context.hip", "actq_linear.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # the scaling step of the quantizer is a separately rounded subtract and multiply
    "-ffp-contract=off",
    # inputs are finite by contract: lets min/max compile to single v_min/v_max (and fold
    # into DPP forms) instead of quieting signalling NaNs first
    "-fno-honor-nans",
    # keep binary32 arithmetic on the scalar-issue VALU forms
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # "#pragma unroll" on loops whose trip count is a template parameter that may be a run-time value
    "-Wno-pass-failed",
]


HOST_LIB = os.path.join(_HERE, "actq_torch.so")
HOST_SOURCE = "actq_torch.cpp"
HOST_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
              "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM"]   # what torch's headers for this platform ask for


def _digest(files, *texts) -> str:
    import hashlib
    h = hashlib.sha256()
    for path in files:
        h.update(os.path.basename(path).encode())
        with open(path, "rb") as f:
            h.update(f.read())
    for text in texts:
        h.update(text.encode())
    return h.hexdigest()[:16]


def source_hash() -> str:
    """Digest of everything the library depends on: the sources, the public and internal headers
    and the compiler flags."""
    files = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC)) if f.endswith((".hip", ".cpp", ".h")) and f != HOST_SOURCE]
    return _digest(files + [os.path.join(ROOT, "include", "actq.h")], " ".join(HIPCC_FLAGS))


def host_source_hash() -> str:
    """The same for the binding's native half, which depends on the interpreter's binary interface and on torch's as well."""
    import sysconfig
    import torch
    return _digest([os.path.join(CSRC, HOST_SOURCE), os.path.join(ROOT, "include", "actq.h")], " ".join(HOST_FLAGS),
                   f"{sysconfig.get_config_var('SOABI')} torch {torch.__version__} {_abi_flag()}")


def _abi_flag() -> str:
    """The C++ library's interface that this torch was built with."""
    import torch
    return f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}"


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found: libactq cannot be built")
    return exe


def build(verbose: bool = False) -> str:
    """Compile every source of the library; always recompiles."""
    tmp = LIB + f".{os.getpid()}.tmp"
    cmd = [hipcc(), *HIPCC_FLAGS, f'-DACTQ_SOURCE_HASH="{source_hash()}"',
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-x", "hip"]
    cmd += [os.path.join(CSRC, s) for s in SOURCES]
    cmd += ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed:\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


def build_host(verbose: bool = False) -> str:
    """Compile the binding's native half; always recompiles."""
    import sysconfig
    import torch
    where = os.path.dirname(torch.__file__)
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        raise RuntimeError("no C++ compiler: actq_torch cannot be built")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc())))
    tmp = HOST_LIB + f".{os.getpid()}.tmp"
    cmd = [cxx, *HOST_FLAGS, f'-DACTQ_SOURCE_HASH="{host_source_hash()}"', _abi_flag()]
    for path in (os.path.join(ROOT, "include"), os.path.join(where, "include"), os.path.join(where, "include", "torch", "csrc", "api", "include"),
                 os.path.join(rocm, "include"), sysconfig.get_paths()["include"]):
        cmd += ["-isystem" if path.startswith(where) else "-I", path]
    cmd += [os.path.join(CSRC, HOST_SOURCE), "-o", tmp, "-L" + os.path.join(where, "lib"), "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch", "-ltorch_python"]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"{cxx} failed:\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    os.replace(tmp, HOST_LIB)
    return HOST_LIB


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_host(verbose=True))
