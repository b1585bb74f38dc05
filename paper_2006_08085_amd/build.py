"""Build libdetag.so (HIP, gfx950 only) in-tree with hipcc, and the binding's native calls (host code) with g++ where
torch and the headers for that are there.

    python -m paper_2006_08085_amd.build [--sanitize-host]

Objects go to _build/ at the repository root; the shared libraries land next to
this file so that they travel with the source tree.
"""
from __future__ import annotations

import glob
import hashlib
import os
import re
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor
from typing import List, Optional

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libdetag.so")
TAG_DIGITS = 12
CALLS_SOURCES = [os.path.join(CSRC, "py_calls.cpp"), os.path.join(ROOT, "include", "detag.h")]

SOURCES = ["topology.cpp", "consensus.cpp", "detag_api.hip", "k_stream.hip", "k_fused.hip", "k_fused_quad.hip", "k_fused_generic.hip", "k_fused_generic_quad.hip",
           "k_diag.hip", "k_grad.hip", "k_softmax.hip", "k_consensus.hip", "k_dense.hip", "k_dense_resident.hip"]

FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-fno-gpu-rdc",
         # packed fp32 VALU forms are kept off for every kernel in this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # the register-resident kernels rely on full unrolling of their row loops (static register indices)
         "-mllvm", "-pragma-unroll-threshold=1000000",
         "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
         "-I", os.path.join(ROOT, "include")]


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found")


# Host-side AddressSanitizer + UndefinedBehaviorSanitizer (the device code is compiled as usual): for running the
# host logic - graph and matrix ingestion, the eigen-solve, the consensus factors, the table builders, argument
# checks - under the sanitizers on a machine without a GPU.
SAN_FLAGS = ["-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
             "-Xarch_host", "-fno-sanitize-recover=undefined", "-Xarch_host", "-fno-omit-frame-pointer"]
SAN_LIB = os.path.join(ROOT, "_build", "san", "libdetag_san.so")


def sanitizer_runtime() -> str:
    """The shared AddressSanitizer runtime of the compiler hipcc drives; a process that loads SAN_LIB into an
    uninstrumented executable (python) must have it in LD_PRELOAD."""
    import glob
    hits = sorted(glob.glob("/opt/rocm/lib/llvm/lib/clang/*/lib/linux/libclang_rt.asan-x86_64.so"))
    if not hits:
        raise RuntimeError("libclang_rt.asan-x86_64.so not found under /opt/rocm/lib/llvm")
    return hits[-1]


def calls_path() -> Optional[str]:
    """Where the native calls are for this interpreter, this torch and these sources: built for another, they have another
    name and are not loaded.  None without torch or the sources."""
    try:
        import torch
        tag = hashlib.sha256(b"".join(open(f, "rb").read() for f in CALLS_SOURCES)).hexdigest()[:TAG_DIGITS]
    except (ImportError, OSError):
        return None
    torch_version = re.sub(r"[^\w.]", "_", torch.__version__)
    return os.path.join(HERE, f"_calls-torch{torch_version}-{tag}{sysconfig.get_config_var('EXT_SUFFIX')}")


def calls_command(source: str, out: str) -> Optional[List[str]]:
    """The command that builds such a module; None where the compiler, torch or the headers it needs are not there."""
    try:
        import torch
    except ImportError:
        return None
    gxx, python_include = shutil.which("g++"), sysconfig.get_paths()["include"]
    torch_dir = os.path.dirname(torch.__file__)
    torch_include = os.path.join(torch_dir, "include")
    if not gxx or not os.path.exists(os.path.join(python_include, "Python.h")) \
            or not os.path.exists(os.path.join(torch_include, "torch", "csrc", "autograd", "python_variable.h")):
        return None
    return [gxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Wno-unknown-pragmas",
            "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", python_include, "-isystem", torch_include,
            "-isystem", os.path.join(torch_include, "torch", "csrc", "api", "include"), source, "-o", out,
            # loaded already, with torch, when this library is
            "-L", os.path.join(torch_dir, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build_calls() -> Optional[str]:
    """Builds the Python calls of the hot path (host code against torch's headers) next to this file.  The binding does
    without them, by ctypes, so what keeps them from being built is reported and no error: returns None then."""
    out = calls_path()
    tmp = f"{out}.{os.getpid()}.tmp"
    cmd = out and calls_command(CALLS_SOURCES[0], tmp)
    if not cmd:
        print("native calls not built: they need g++, torch with its headers and Python's", file=sys.stderr)
        return None
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        print(f"native calls not built: g++ failed on {CALLS_SOURCES[0]}:\n{r.stdout}{r.stderr}", file=sys.stderr)
        return None
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    for other in glob.glob(out[:-len(suffix) - TAG_DIGITS] + "*" + suffix):  # of other sources
        if other != out:
            os.remove(other)
    os.replace(tmp, out)
    return out


def ensure_built() -> None:
    """Builds what the binding loads and is not there."""
    from .binding import LIB_PATH
    if not os.path.exists(LIB_PATH):
        build(verbose=False)
    elif LIB_PATH == LIB and calls_path() and not os.path.exists(calls_path()):
        build_calls()


def build(verbose: bool = True, jobs: int = 8, sanitize_host: bool = False) -> str:
    """Builds libdetag.so and the native calls next to this file; with sanitize_host the instrumented SAN_LIB under _build/san instead
    (load it with DETAG_LIB=<path> and LD_PRELOAD=sanitizer_runtime())."""
    hipcc = _hipcc()
    bdir = os.path.join(ROOT, "_build", "san") if sanitize_host else os.path.join(ROOT, "_build")
    os.makedirs(bdir, exist_ok=True)
    srcs = list(SOURCES)
    extra = SAN_FLAGS if sanitize_host else []
    link_extra = ["-fsanitize=address", "-fsanitize=undefined", "-shared-libsan", "-Wno-option-ignored"] if sanitize_host else []

    def compile_one(src: str) -> str:
        obj = os.path.join(bdir, src + ".o")
        cmd = [hipcc, *FLAGS, *extra, "-I", CSRC, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        out = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                        if "packed-fp32-ops" not in l and "is not a recognized feature" not in l)
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out, file=sys.stderr)
        return obj

    with ThreadPoolExecutor(max_workers=jobs) as ex:
        if not sanitize_host:
            ex.submit(build_calls)
        objs = list(ex.map(compile_one, srcs))
    lib_out = SAN_LIB if sanitize_host else LIB
    tmp = lib_out + ".tmp"
    r = subprocess.run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-fno-gpu-rdc", *link_extra, "-o", tmp, *objs],
                       capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n" + r.stdout + r.stderr)
    os.replace(tmp, lib_out)
    if verbose:
        print(f"built {lib_out}")
    return lib_out


if __name__ == "__main__":
    build(sanitize_host="--sanitize-host" in sys.argv[1:])
