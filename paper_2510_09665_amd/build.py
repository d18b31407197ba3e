"""Builds liblmc.so (HIP kernels + C ABI) for gfx950 with hipcc and the Python extension module
over it with the host compiler, in-tree.

hipcc cross-compiles without a GPU.  Run as `python -m paper_2510_09665_amd.build`.
"""
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblmc.so")
EXTENSION = os.path.join(HERE, "_lmc_native.so")
EXTENSION_SOURCE = os.path.join(CSRC, "lmc_py.cpp")
SOURCES = ["lmc_kernels.hip", "lmc_ctx.cpp", "lmc_pipeline.cpp", "lmc_streams.cpp", "lmc_measure.cpp", "lmc_static.cpp",
           "lmc_seq.cpp", "lmc_window.cpp", "lmc_tier.cpp"]
HEADERS = ["lmc_ctx.hpp", "lmc_kernels.hpp", "lmc_index.hpp", "lmc_window.hpp", "lmc_guard.hpp", os.path.join("..", "..", "include", "lmc.h")]

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-x", "hip",
    "-Wall", "-Wextra", "-Wno-unused-parameter",
    # keep the compiler from forming packed-fp32 instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def stale():
    if not os.path.exists(LIB) or not os.path.exists(EXTENSION):
        return True
    t = min(os.path.getmtime(LIB), os.path.getmtime(EXTENSION))
    return any(os.path.getmtime(os.path.join(CSRC, f)) > t for f in SOURCES + HEADERS + [EXTENSION_SOURCE])


def _compile(cmd, out, verbose):
    tmp = out + ".%d.tmp" % os.getpid()
    cmd = cmd + ["-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the gfx950 target feature and says so: harmless
    said = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("%s failed:\n%s" % (cmd[0], said))
    if verbose and said.strip():
        print(said)
    os.replace(tmp, out)


def build(force=True, verbose=False):
    """Compile every source into liblmc.so, and the extension module; returns the library's path."""
    if not force and not stale():
        return LIB
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    _compile([hipcc] + FLAGS + [os.path.join(CSRC, s) for s in SOURCES], LIB, verbose)
    _compile([os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wextra",
              "-I" + sysconfig.get_paths()["include"], EXTENSION_SOURCE, "-ldl"], EXTENSION, verbose)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
