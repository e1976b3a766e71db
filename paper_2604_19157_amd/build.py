"""Compile the HIP sources in ``csrc/`` into ``libsaw.so`` for gfx950 (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import glob
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libsaw.so")
MARSHAL = os.path.join(HERE, "_marshal.so")     # the binding's argument marshalling (csrc/marshal.cpp)

HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC",
    # packed fp32 VALU ops are switched off for every kernel of this library
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

# per-source additions
EXTRA_FLAGS = {
    # MFMA results stay in ordinary VGPRs (no accumulator-register copies around the matrix ops)
    "saw_store_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
    "saw_flatten.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
}


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + r.stdout + r.stderr)


def build_library(verbose: bool = False) -> str:
    """Always recompiles every source; returns the path of the shared library."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(HERE, "csrc")]
    objs = []
    procs = []
    for src in sources():
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        cmd = ["hipcc", *HIPCC_FLAGS, *EXTRA_FLAGS.get(os.path.basename(src), []), *inc, "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((cmd, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True)))
        objs.append(obj)
    for cmd, pr in procs:
        out, err = pr.communicate()
        if pr.returncode != 0:
            raise RuntimeError("hipcc failed: " + " ".join(cmd) + "\n" + out + err)
    _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB + ".tmp", *objs], verbose)
    os.replace(LIB + ".tmp", LIB)
    build_marshal(verbose)
    return LIB


def build_marshal(verbose: bool = False) -> str | None:
    """Host code only: a Python extension module against torch's headers, linked to ``libsaw.so`` beside it.  Where those headers or
    Python's are not installed there is none, and the binding goes through ctypes."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    inc = [os.path.join(ROOT, "include"), os.path.join(t, "include"), os.path.join(t, "include", "torch", "csrc", "api", "include"),
           os.path.join(rocm, "include"), sysconfig.get_paths()["include"]]
    if not (os.path.exists(os.path.join(inc[-1], "Python.h")) and os.path.exists(os.path.join(inc[1], "torch"))):
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)                  # (an older one would not fit the library)
        print("no headers of Python and torch: _marshal.so is not built", flush=True)
        return None
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
          f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *["-I" + d for d in inc],
          os.path.join(HERE, "csrc", "marshal.cpp"), "-o", MARSHAL + ".tmp", "-L" + HERE, "-l:libsaw.so", "-Wl,-rpath,$ORIGIN",
          "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"], verbose)
    os.replace(MARSHAL + ".tmp", MARSHAL)
    return MARSHAL


if __name__ == "__main__":
    print(build_library(verbose=True))
