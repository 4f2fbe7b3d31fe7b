"""Build librapid_attn.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SOURCES = [os.path.join(HERE, "csrc", "rapid_attn.hip"), os.path.join(HERE, "csrc", "rapid_cache.hip"),
           os.path.join(HERE, "csrc", "rapid_mask.hip")]
OUT = os.path.join(HERE, "librapid_attn.so")
# measurement aid used by bench.py only (an MFMA-only loop), kept out of the attention library
PROBE_SOURCES = [os.path.join(HERE, "csrc", "mfma_probe.hip")]
PROBE_OUT = os.path.join(HERE, "libmfma_probe.so")

# the launching entry points called with tensors (host code; see its head)
NATIVE_SOURCE = os.path.join(HERE, "csrc", "native_call.cpp")
NATIVE_OUT = os.path.join(HERE, "native_call.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-fvisibility=hidden", "-fno-gpu-rdc",
    # no HIP runtime is linked in: the library binds to the libamdhip64 already loaded
    # in the process (PyTorch's), so streams and pointers belong to the same runtime
    "-no-hip-rt",
    # packed fp32 VALU forms are kept off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"),
]


def build(verbose: bool = False, extra: list[str] | None = None, out: str = OUT) -> str:
    _compile(PROBE_SOURCES, PROBE_OUT, verbose, extra)
    _compile(SOURCES, out, verbose, extra)
    build_native(verbose)
    return out


def native_lacks() -> str | None:
    """What a compilation of native_call.so would need and is not here, or None."""
    import sysconfig
    if shutil.which("g++") is None:
        return "g++"
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return "Python.h"
    try:
        from torch.utils.cpp_extension import include_paths
    except ImportError:
        return "torch"
    header = os.path.join("torch", "csrc", "autograd", "python_variable.h")
    return None if any(os.path.exists(os.path.join(path, header)) for path in include_paths()) else header


def build_native(verbose: bool = False) -> str | None:
    """native_call.so; None where it cannot be compiled: the calls then go by way of ctypes."""
    lacks = native_lacks()
    if lacks is not None:
        print(f"{NATIVE_OUT} is not built ({lacks} is missing): calls go by way of ctypes", file=sys.stderr)
        if os.path.exists(NATIVE_OUT):
            os.remove(NATIVE_OUT)                 # of other sources
        return None
    import sysconfig

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           f'-DBUILT_FOR="{torch.__version__} {sys.implementation.cache_tag}"',
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", os.path.join(ROOT, "include")]
    for path in include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", path]
    for path in library_paths():
        cmd += ["-L", path]
    return _run(cmd + ["-o", NATIVE_OUT, NATIVE_SOURCE, "-ltorch_python", "-ltorch_cpu", "-lc10"], NATIVE_OUT, verbose)


def _compile(sources, out, verbose, extra):
    return _run([HIPCC] + FLAGS + (extra or []) + ["-o", out] + sources, out, verbose)


def _run(cmd, out, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "packed-fp32-ops"
    err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed ({res.returncode}):\n{err}")
    if verbose and err.strip():
        print(err, file=sys.stderr)
    return out


if __name__ == "__main__":
    print(build(verbose=True))
