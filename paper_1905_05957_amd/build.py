"""Builds, in tree, libds_hip.so (the C-ABI library of HIP kernels, for gfx950 with hipcc) and _fastcall.so (the
Python binding's step calls, host code only)."""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libds_hip.so")
FASTCALL, FASTCALL_SRC = os.path.join(HERE, "_fastcall.so"), os.path.join(CSRC, "fastcall.cpp")
SOURCES = ["ds_api.hip", "identity.hip", "sign.hip", "qsgd.hip", "topk.hip", "clip.hip", "rsparse.hip", "ternary.hip"]
HEADERS = ["ds_device.h", "held.h", "ds_internal.h", os.path.join("..", "..", "include", "ds.h")]

# -ffp-contract=off: every fused multiply-add in the kernels is an explicit __fmaf_rn, so
#   results do not depend on the compiler's contraction choices.
# -packed-fp32-ops off: the compiler must not form packed fp32 instructions.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
    "-fhip-fp32-correctly-rounded-divide-sqrt", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def build_fastcall(force: bool = True) -> str:
    """Compile the binding's extension module against this interpreter and its torch."""
    deps = [FASTCALL_SRC, os.path.normpath(os.path.join(CSRC, "..", "..", "include", "ds.h"))]
    if not force and os.path.exists(FASTCALL) and all(os.path.getmtime(FASTCALL) >= os.path.getmtime(p) for p in deps):
        return FASTCALL
    import sysconfig
    import torch
    base = os.path.dirname(torch.__file__)
    tmp = FASTCALL + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), "-isystem", os.path.join(base, "include"),
           "-isystem", sysconfig.get_paths()["include"], FASTCALL_SRC, "-o", tmp, "-L" + os.path.join(base, "lib"),
           "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("compilation of _fastcall.so failed")
    os.replace(tmp, FASTCALL)
    return FASTCALL


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every source, link the shared library and build the extension module.  Always recompiles when force."""
    with ThreadPoolExecutor(max_workers=1) as ex:
        fastcall = ex.submit(build_fastcall, force)
        lib = build_library(force, verbose)
        fastcall.result()
    return lib


def build_library(force: bool = True, verbose: bool = False) -> str:
    """Compile the HIP sources and link libds_hip.so."""
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    deps = srcs + [os.path.normpath(os.path.join(CSRC, h)) for h in HEADERS]
    if not force and os.path.exists(LIB) and all(os.path.getmtime(LIB) >= os.path.getmtime(p) for p in deps):
        return LIB
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    hipcc = _hipcc()

    def compile_one(src: str) -> str:
        obj = os.path.join(objdir, os.path.basename(src) + ".o")
        cmd = [hipcc, *HIPCC_FLAGS, *os.environ.get("DS_EXTRA_HIPCC_FLAGS", "").split(), "-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            sys.stderr.write(r.stdout + r.stderr)
            raise RuntimeError(f"hipcc failed on {src}")
        noise = "'-packed-fp32-ops' is not a recognized feature"
        err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
        if verbose and err.strip():
            sys.stderr.write(err + "\n")
        return obj

    with ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(compile_one, srcs))
    tmp = LIB + ".tmp%d" % os.getpid()
    r = subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link of libds_hip.so failed")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose="-v" in sys.argv))
