"""Builds and runs hipstub.cpp: the library's host code over a HIP runtime in
host memory (test infrastructure)."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.join(HERE, "..", "..")
EXE = os.path.join(HERE, "_build", "hipstub")


def run(scenario: str) -> list[list[str]]:
    """The words of each line that the scenario prints."""
    from paper_2007_00324_amd import gdp2d
    from paper_2007_00324_amd.build import CSRC, HIPCC, LIB
    gdp2d.load()  # (built by now)
    src = os.path.join(HERE, "hipstub.cpp")
    deps = [src, os.path.join(CSRC, "gdp_internal.h"), os.path.join(ROOT, "include", "gdp2d.h"), LIB]
    if not os.path.exists(EXE) or os.path.getmtime(EXE) < max(os.path.getmtime(d) for d in deps):
        os.makedirs(os.path.dirname(EXE), exist_ok=True)
        tmp = f"{EXE}.{os.getpid()}"  # test workers may build at the same time
        subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                        "-o", tmp, src, "-L", os.path.dirname(LIB), "-l:" + os.path.basename(LIB),
                        "-Wl,-rpath," + os.path.dirname(LIB), "-rdynamic", "-lpthread", "-ldl"], check=True, capture_output=True)
        os.replace(tmp, EXE)
    r = subprocess.run([EXE, scenario], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stdout, r.stderr)
    return [line.split() for line in r.stdout.splitlines()]
