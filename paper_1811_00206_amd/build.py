"""Build ``libbs.so``, ``_native.so`` and ``libbs_probe.so`` in-tree for gfx950.

``python -m paper_1811_00206_amd.build`` compiles every ``csrc/*.hip`` into the
product library ``libbs.so``, ``csrc/bs_calls.cpp`` (host code: the marshalling
of the Python calls, against torch's headers) into the extension module
``_native.so``, and every ``probe/*.hip`` (measurement helpers for the
benchmark, not part of the method) into ``libbs_probe.so``, all next to this
file.  Cross-compilation needs no GPU.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
PROBE_SRC = os.path.join(HERE, "probe")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libbs.so")
PROBE_LIB = os.path.join(HERE, "libbs_probe.so")
NATIVE_SRC = os.path.join(CSRC, "bs_calls.cpp")
NATIVE_LIB = os.path.join(HERE, "_native.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed fp32 instructions are kept off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    # an unrolled loop with an early exit is unrolled by a later pass than the one that warns
    "-Wno-pass-failed",
]


def is_built() -> bool:
    """Whether what the calls load is there: the library and the native marshalling beside it."""
    return os.path.exists(LIB) and os.path.exists(NATIVE_LIB)


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def probe_sources():
    return sorted(glob.glob(os.path.join(PROBE_SRC, "*.hip")))


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
    subprocess.check_call([HIPCC, *FLAGS, "-c", src, "-o", obj])
    return obj


def _link(lib: str, objs) -> None:
    tmp = lib + f".tmp{os.getpid()}"
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, lib)


def native_compiler():
    """The host compiler and its flags for code against torch's headers."""
    import torch
    from torch.utils import cpp_extension
    inc = [*cpp_extension.include_paths(), sysconfig.get_paths()["include"], "/opt/rocm/include"]
    return [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
            "-DUSE_ROCM", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
            *(f"-isystem{d}" for d in inc)]


def _compile_native() -> str:
    obj = os.path.join(OBJDIR, "bs_calls.cpp.o")
    subprocess.check_call([*native_compiler(), "-c", NATIVE_SRC, "-o", obj])
    return obj


def _link_native(obj: str) -> None:
    # torch's libraries are loaded when this module is; libbs.so lies beside it
    import torch
    tmp = NATIVE_LIB + f".tmp{os.getpid()}"
    subprocess.check_call([os.environ.get("CXX", "g++"), "-shared", "-o", tmp, obj,
                           "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu",
                           "-lc10", "-lc10_hip", "-L" + HERE, "-l:libbs.so", "-Wl,-rpath,$ORIGIN"])
    os.replace(tmp, NATIVE_LIB)


def build_library(verbose: bool = False) -> str:
    """Compile all sources (always; no staleness shortcut) and link libbs.so, _native.so
    and libbs_probe.so."""
    os.makedirs(OBJDIR, exist_ok=True)
    srcs, psrcs = sources(), probe_sources()
    if not srcs:
        raise RuntimeError("no HIP sources found under " + CSRC)
    jobs = max(1, min(len(srcs) + len(psrcs) + 1, 8, os.cpu_count() or 1))
    with ThreadPoolExecutor(jobs) as ex:
        native = ex.submit(_compile_native)
        objs = list(ex.map(_compile, srcs + psrcs))
    _link(LIB, objs[:len(srcs)])
    _link_native(native.result())
    if psrcs:
        _link(PROBE_LIB, objs[len(srcs):])
    if verbose:
        print("built", LIB + ",", NATIVE_LIB, "and", PROBE_LIB)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
    sys.exit(0)
