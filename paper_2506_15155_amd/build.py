"""Build libellm.so (HIP, gfx950) in-tree with hipcc, and _calls, the native part of the Python binding, with g++."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libellm.so")
# (named for the interpreter it is built for: another one does not load it)
CALLS = os.path.join(HERE, "_calls" + sysconfig.get_config_var("EXT_SUFFIX"))
CALLS_SOURCE = os.path.join(CSRC, "python_calls.cpp")
SOURCES = ["pool_core.cpp", "ellm_api.cpp", "kernels.hip"]
HEADERS = ["pool_core.hpp", "kernels.hpp", "divide.hpp", "map_queue.hpp", os.path.join(ROOT, "include", "ellm.h")]

# packed-fp32 instructions are switched off for all device code of this library
DEVICE_FLAGS = ["-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def needs_build() -> bool:
    if not os.path.exists(LIB) or not os.path.exists(CALLS) or os.path.getmtime(CALLS_SOURCE) > os.path.getmtime(CALLS):
        return True
    t = os.path.getmtime(LIB)
    deps = [os.path.join(CSRC, s) for s in SOURCES] + [h if os.path.isabs(h) else os.path.join(CSRC, h) for h in HEADERS]
    return any(os.path.getmtime(d) > t for d in deps)


def build(force: bool = True, verbose: bool = False) -> str:
    if not force and not needs_build():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall",
           "-Wno-unused-result", *DEVICE_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC,
           *[os.path.join(CSRC, s) for s in SOURCES], "-o", LIB]
    import numpy
    calls = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", sysconfig.get_paths()["include"],
             "-I", numpy.get_include(), CALLS_SOURCE, "-o", CALLS]
    for c in (cmd, calls):
        if verbose:
            print(" ".join(c))
        subprocess.run(c, check=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
