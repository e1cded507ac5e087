"""Build the HIP shared library for gfx950 with hipcc (no JIT, in-tree output)."""
from __future__ import annotations

import os
import subprocess
import sysconfig
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libscout.so")
SOURCES = ["score.hip", "append.hip", "fetch.hip", "topk.hip", "attn.hip", "api.hip"]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    # keep hipcc from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
]


CALIB_LIB = os.path.join(HERE, "libscout_calib.so")


def _run(cmd, verbose):
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(ln for ln in res.stderr.splitlines() if noise not in ln)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + err)
    if verbose and err.strip():
        print(err)


def _hipcc(sources, out, verbose):
    """Every source to an object of its own (in parallel: the kernels share no device symbols), then one link."""
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(max_workers=4) as pool:
        objs = [os.path.join(tmp, s + ".o") for s in sources]
        compile_flags = [f for f in FLAGS if f != "-shared"]
        list(pool.map(lambda so: _run(["hipcc", *compile_flags, *inc, "-c", os.path.join(CSRC, so[0]), "-o", so[1]], verbose),
                      zip(sources, objs)))
        _run(["hipcc", "--offload-arch=gfx950", "-fPIC", "-shared", *objs, "-o", out], verbose)
    return out


def build(verbose: bool = False) -> str:
    """Compile every kernel source into libscout.so next to this file (the measurement aids into
    libscout_calib.so, a library of their own, and the Python entry points into _calls.so); returns the path of
    libscout.so."""
    build_calls(verbose)
    _hipcc(["calib.hip"], CALIB_LIB, verbose)
    return _hipcc(SOURCES, LIB, verbose)


# the entry points as Python functions on torch tensors (CPython extension)
CALLS_LIB = os.path.join(HERE, "_calls.so")


def build_calls(verbose: bool = False) -> str:
    """Compile the argument marshalling (plain C++17 against the installed torch's headers) into _calls.so."""
    import torch
    tdir = os.path.dirname(torch.__file__)
    inc = [os.path.join(ROOT, "include"), sysconfig.get_paths()["include"], os.path.join(tdir, "include"),
           os.path.join(tdir, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include"]
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *[f"-I{i}" for i in inc],
          os.path.join(CSRC, "py_calls.cpp"), "-o", CALLS_LIB, "-L", os.path.join(tdir, "lib"),
          "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_python"], verbose)
    return CALLS_LIB


HOST_LIB = os.path.join(HERE, "libscout_host.so")


def build_host(verbose: bool = False) -> str:
    """Compile the host-side worker (plain C++17, threads) into libscout_host.so next to this file."""
    cmd = ["g++", "-O3", "-std=c++17", "-fPIC", "-shared", "-pthread", "-Wall", "-Wextra", "-Wno-psabi",
           "-I", os.path.join(ROOT, "include"), os.path.join(CSRC, "host_worker.cpp"), "-o", HOST_LIB]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n" + res.stderr)
    if verbose and res.stderr.strip():
        print(res.stderr)
    return HOST_LIB


if __name__ == "__main__":
    print(build(verbose=True))
    print(build_host(verbose=True))
