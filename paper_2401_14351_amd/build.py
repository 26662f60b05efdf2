"""Build ``libsllm.so`` in-tree: the C++ host runtime and the gfx950 HIP kernels
behind the C ABI declared in ``include/sllm.h``; and ``_views``, the Python
binding's native view builder, the only part that knows torch: left out, with a
note, where torch or its headers are not installed.

Run ``python -m paper_2401_14351_amd.build`` (or ``__graft_entry__.build()``).
"""

from __future__ import annotations

import os
import shlex
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
OBJDIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libsllm.so")
VIEWS_SRC = os.path.join(PKG, "pyext", "views.cpp")
VIEWS = os.path.join(PKG, "_views" + sysconfig.get_config_var("EXT_SUFFIX"))  # names the Python it is for
ARCH = "gfx950"

# Every HIP compile leaves packed-FP32 instructions out of the generated code.
HIP_FLAGS = ["-x", "hip", f"--offload-arch={ARCH}", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")
COMMON = ["-O3", "-fPIC", "-std=c++17", "-Wall", "-Wextra", "-Wno-unused-parameter", f"-I{INCLUDE}", f"-I{CSRC}"]
# host-only sources: plain C++ against the HIP runtime headers
HOST_FLAGS = [f"-I{ROCM}/include", "-D__HIP_PLATFORM_AMD__"]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".cpp", ".hip")))


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def _cxx() -> str:
    return os.environ.get("CXX", "g++")


def _run(cmd, verbose):
    if verbose:
        print(" ".join(shlex.quote(c) for c in cmd), flush=True)
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # hipcc's host pass does not know the packed-fp32 feature; that note is expected
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError(f"build failed: {' '.join(cmd)}\n{out}")
    if verbose and out.strip():
        print(out, flush=True)


def views_command(out: str):
    """The compiler call that makes the view builder for this interpreter and
    its torch, or None without torch's headers."""
    try:
        import torch
    except ImportError:
        return None
    base = os.path.dirname(os.path.abspath(torch.__file__))
    inc = [os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include")]
    python = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(inc[0], "ATen", "Functions.h")) or not os.path.exists(os.path.join(python, "Python.h")):
        return None
    return [_cxx(), "-shared", "-O2", "-fPIC", "-std=c++17", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch.compiled_with_cxx11_abi())}",
            f"-I{INCLUDE}", *[a for i in inc for a in ("-isystem", i)], f"-I{python}", VIEWS_SRC,
            "-o", out, f"-L{os.path.join(base, 'lib')}", "-ltorch_python", "-ltorch_cpu", "-lc10"]


def build(verbose: bool = False) -> str:
    """Compile every source, link ``libsllm.so`` and the view builder; return the former's path."""
    os.makedirs(OBJDIR, exist_ok=True)
    jobs = []
    for src in sources():
        obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
        if src.endswith(".hip"):
            cmd = [_hipcc(), "-c", *COMMON, *HIP_FLAGS, src, "-o", obj]
        else:
            cmd = [_cxx(), "-c", *COMMON, *HOST_FLAGS, src, "-o", obj]
        jobs.append((cmd, obj))
    views_tmp = VIEWS + ".tmp"
    views = views_command(views_tmp)
    if views:
        jobs.insert(0, (views, None))  # the longest one first
    else:
        print("no torch headers: the view builder is left out, views are built in Python", flush=True)
    workers = max(1, min(len(jobs), os.cpu_count() or 1, 16))
    with ThreadPoolExecutor(workers) as ex:
        list(ex.map(lambda j: _run(j[0], verbose), jobs))
    tmp = LIB + ".tmp"
    _run([_hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", *[o for _, o in jobs if o], "-o", tmp, "-lpthread"], verbose)
    os.replace(tmp, LIB)
    if views:
        os.replace(views_tmp, VIEWS)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
