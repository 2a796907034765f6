"""Builds libheinsen.so (HIP, gfx950) in-tree with hipcc.  Usage: python -m paper_2311_06281_amd.build"""
from __future__ import annotations

import os
import shlex
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libheinsen.so")
SOURCES = ["heinsen_api.hip", "scan_bnd.hip", "scan_bdn.hip", "sequential_ref.hip", "stream_probe.hip"]
HEADERS = ["heinsen_internal.hpp", "heinsen_math.hpp", "heinsen_tickets.hpp", "scan_rules.hpp", os.path.join("..", "..", "include", "heinsen.h")]
CALL_SOURCE = "call.c"  # the Python side of the scan entry points
CALL = os.path.join(HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CC = shlex.split(os.environ.get("CC", "gcc"))
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-command-line-argument",
         # packed-FP32 instructions are kept out of the generated code
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def _compile(src: str) -> str:
    obj = os.path.join(CSRC, os.path.splitext(src)[0] + ".o")
    extra = os.environ.get("HEINSEN_EXTRA_HIPCC_FLAGS", "").split()  # extra compiler flags for development builds
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_call() -> None:
    """The call module.  Without it (no C compiler, no Python headers) the binding converts every argument in Python."""
    include = sysconfig.get_paths()["include"]
    cmd = [*CC, "-O2", "-Wall", "-shared", "-fPIC", "-I", include, os.path.join(CSRC, CALL_SOURCE), "-o", CALL]
    try:
        r = subprocess.run(cmd, capture_output=True, text=True)
        failed, why = r.returncode != 0, r.stderr
    except OSError as e:
        failed, why = True, f"{e}\n"
    if failed:
        if os.path.exists(CALL):
            os.remove(CALL)  # of another build
        sys.stderr.write(f"{CALL_SOURCE} was not compiled, calls from Python take about 1.1 us longer:\n{why}")


def _older(built: str, sources: list) -> bool:
    return not os.path.exists(built) or any(os.path.getmtime(os.path.join(CSRC, s)) > os.path.getmtime(built) for s in sources)


def needs_build() -> bool:
    return _older(LIB, SOURCES + HEADERS)


def build(force: bool = True) -> str:
    """Compile every translation unit and link the shared library, then the call module. Returns the library's path."""
    if force or needs_build():
        with ThreadPoolExecutor(max_workers=len(SOURCES)) as ex:
            objs = list(ex.map(_compile, SOURCES))
        cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError(f"link failed:\n{r.stderr}")
    if force or _older(CALL, [CALL_SOURCE]):
        _compile_call()
    return LIB


if __name__ == "__main__":
    print(build())
