"""Rounds of the Flip-Flop insertion on the host (tests.ffemu) whose removal
passes run the kernels' own text lane by lane (test infrastructure).

ff_round.cpp is built with hipcc as plain host code, ff_lanes.cpp, which
includes gdp_ff.hip, as plain C++."""
from __future__ import annotations

import ctypes as C
import os
import subprocess

from tests import ffemu

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(HERE, "libfflanes.so")
_lib = None


def _build() -> None:
    tmp = f"{LIB}.{os.getpid()}.tmp"  # test workers may build at the same time
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(hipcc)))
    flags = ["-O2", "-std=c++17", "-fPIC", "-ffp-contract=off", "-fno-fast-math", "-I", ffemu.CORE]
    for cmd in ([os.path.join(rocm, "llvm", "bin", "clang++"), "-x", "c++", *flags, "-D__HIP_PLATFORM_AMD__", "-w",
                 "-I", os.path.join(rocm, "include"), "-c", "-o", f"{tmp}.1.o", os.path.join(HERE, "ff_lanes.cpp")],
                [hipcc, *flags, "-c", "-o", f"{tmp}.2.o", os.path.join(HERE, "ff_round.cpp")],
                [hipcc, "-shared", "-o", tmp, f"{tmp}.1.o", f"{tmp}.2.o"]):
        subprocess.run(cmd, check=True, capture_output=True)
    os.remove(f"{tmp}.1.o")
    os.remove(f"{tmp}.2.o")
    os.replace(tmp, LIB)


def load():
    global _lib
    if _lib is None:
        srcs = [os.path.join(HERE, f) for f in ("ff_lanes.cpp", "ff_round.cpp", "__init__.py")]
        srcs += [os.path.join(ffemu.HERE, "ff_emu.cpp")]
        srcs += [os.path.join(ffemu.CORE, f) for f in ("gdp_ff_core.h", "gdp_exact.h", "gdp_ff.hip", "gdp_kernels.h",
                                                       "gdp_internal.h")]
        if not os.path.exists(LIB) or os.path.getmtime(LIB) < max(os.path.getmtime(s) for s in srcs):
            _build()
        _lib = C.CDLL(LIB)
        _lib.ffemu_round.argtypes = ffemu.load().ffemu_round.argtypes
        _lib.ffemu_round.restype = C.c_int32
    return _lib


def links() -> list[int]:
    """Points taken into the passes so far: with a link of a group's size, a wave's, more."""
    return list((C.c_int64 * 3).in_dll(load(), "ffemu_links"))


def round_from_points(*args, **kw):
    """ffemu.round_from_points with the removals by the kernels' text."""
    ffemu.load()
    plain, ffemu._lib = ffemu._lib, load()
    try:
        return ffemu.round_from_points(*args, **kw)
    finally:
        ffemu._lib = plain
