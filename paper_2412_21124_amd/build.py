"""Build ``libnormtest.so`` from ``csrc/normtest.hip`` for gfx950 with hipcc (works without a GPU), and the binding's native call
path from ``csrc/callpath.cpp`` with g++."""
from __future__ import annotations

import os
import subprocess
import sysconfig

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
SRC = os.path.join(_HERE, "csrc", "normtest.hip")
LIB = os.path.join(_HERE, "libnormtest.so")
INCLUDE = os.path.join(ROOT, "include")
CALLPATH_SRC = os.path.join(_HERE, "csrc", "callpath.cpp")

# contraction off: the error-free transformations of the finalize kernel, and the bits that the copies of a tile's
# code (whole and part tiles, every launch shape) have in common, rely on every fused multiply-add being an explicit one;
# packed fp32 instructions are disabled for the device pass.
HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-shared", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def build_library(out: str = LIB, quiet: bool = True) -> str:
    cmd = ["hipcc", *HIPCC_FLAGS, "-I", INCLUDE]
    tmp = out + ".tmp.%d" % os.getpid()
    cmd += ["-o", tmp, SRC]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n%s\n%s" % (" ".join(cmd), res.stderr))
    if not quiet:
        # the host pass does not know the device-only target feature and says so: harmless
        print("\n".join(l for l in res.stderr.splitlines() if "packed-fp32-ops" not in l))
    os.replace(tmp, out)
    return out


def callpath_file() -> str:
    """Where the native call path is built: it fits one Python and one torch, so the name says which."""
    import torch
    return os.path.join(_HERE, "_callpath.torch-%s%s" % (torch.__version__, sysconfig.get_config_var("EXT_SUFFIX")))


def build_callpath() -> str:
    import torch
    from torch.utils.cpp_extension import include_paths
    out = callpath_file()
    tmp = out + ".tmp.%d" % os.getpid()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I", INCLUDE]
    for path in [*include_paths(), sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", path]
    cmd += ["-o", tmp, CALLPATH_SRC, "-L" + os.path.join(os.path.dirname(torch.__file__), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("g++ failed:\n%s\n%s" % (" ".join(cmd), res.stderr))
    os.replace(tmp, out)
    return out


def _stale(built: str, *sources: str) -> bool:
    return not os.path.exists(built) or os.path.getmtime(built) < max(os.path.getmtime(s) for s in sources)


def ensure_built() -> str:
    """Path of the built library; builds it if nothing is there or a source is newer than the build."""
    header = os.path.join(INCLUDE, "normtest.h")
    if _stale(LIB, SRC, header):
        build_library()
    return LIB


def ensure_callpath() -> str:
    """The same for the binding's native part."""
    built = callpath_file()
    if _stale(built, CALLPATH_SRC, os.path.join(INCLUDE, "normtest.h")):
        build_callpath()
    return built


if __name__ == "__main__":
    print(build_library(quiet=False))
    print(build_callpath())
