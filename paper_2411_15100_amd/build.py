"""Build libxgm.so (host C++ + HIP kernels for gfx950) with hipcc and the extension _native of the Python binding
with the host compiler, both in-tree.  The extension's file name carries the tag of the Python it was built for, so
that another one asks for its own instead of loading it."""

from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libxgm.so")
EXT = os.path.join(HERE, "_native" + sysconfig.get_config_var("EXT_SUFFIX"))
EXT_UNTAGGED = os.path.join(HERE, "_native.so")  # (any Python would load it)
EXT_SOURCE = os.path.join(CSRC, "pybinding.cpp")
SOURCES = ["automaton.cpp", "engine.cpp", "schema.cpp", "api.cpp", "kernels.hip"]
HEADERS = ["automaton.hpp", "engine.hpp", "schema.hpp", "kernels.hpp", "walk.hpp", os.path.join("..", "..", "include", "xgm.h")]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Wall", "-Wno-unused-function",
    # packed FP32 instructions are kept off for every kernel
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def _stale(out: str, deps) -> bool:
    return not os.path.exists(out) or os.path.getmtime(out) < max(os.path.getmtime(d) for d in deps)


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + proc.stdout + proc.stderr)
    if verbose and proc.stderr:
        print(proc.stderr, file=sys.stderr)


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source; returns the path of the shared library."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    if force or _stale(LIB, srcs + [os.path.join(CSRC, h) for h in HEADERS]):
        _run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + FLAGS + srcs + ["-o", LIB], verbose)
    if os.path.exists(EXT_UNTAGGED):
        os.remove(EXT_UNTAGGED)
    if force or _stale(EXT, [EXT_SOURCE]):
        _run([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-fvisibility=hidden",
              "-I" + sysconfig.get_paths()["include"], EXT_SOURCE, "-o", EXT], verbose)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
