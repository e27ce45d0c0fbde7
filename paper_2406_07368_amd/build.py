"""Builds liblinattn.so (HIP, gfx950 only) and the extension module of the tensor-level calls next to this file.

    python -m paper_2406_07368_amd.build

hipcc cross-compiles without a GPU.  Packed-fp32 instruction selection is
switched off for all device code.
"""
from __future__ import annotations

import contextlib
import glob
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblinattn.so")
CALLS = os.path.join(HERE, "_calls.so")
CALLS_KEY = os.path.join(HERE, "_calls.key")    # what CALLS was built from and for
OBJ = os.path.join(HERE, "_build")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the device-only feature flag and says so; drop that line
    log = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(f"{cmd[0]} failed:\n" + log)
    if verbose and log.strip():
        print(log)


def calls_key() -> str:
    """The sources of the extension module and the torch and Python it is built for."""
    import hashlib

    import torch

    h = hashlib.sha256(f"{torch.__version__} {torch.version.git_version} {sys.implementation.cache_tag}".encode())
    for path in (os.path.join(CSRC, "calls.cpp"), os.path.join(os.path.dirname(HERE), "include", "linattn.h")):
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def calls_current() -> bool:
    """Whether the extension module that lies there is the one that build_calls would make."""
    try:
        with open(CALLS_KEY) as f:
            return f.read() == calls_key() and os.path.exists(CALLS)
    except FileNotFoundError:
        return False


def build_calls(verbose: bool = False) -> str:
    """csrc/calls.cpp: host code on torch's C++ interface.  Compiled under another name and put in place whole: several
    processes may start at once, and one that finds the file loads it."""
    import sysconfig
    import threading

    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    tmp = f"{CALLS}.{os.getpid()}.{threading.get_ident()}"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           *[f"-isystem{p}" for p in (*include_paths(), sysconfig.get_paths()["include"])], os.path.join(CSRC, "calls.cpp"), "-o", tmp,
           *[f"-L{p}" for p in library_paths()], "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10"]
    key = calls_key()
    try:
        _run(cmd, verbose)
        with contextlib.suppress(FileNotFoundError):
            os.remove(CALLS_KEY)                   # (at no time a key beside a module that is not its own)
        os.replace(tmp, CALLS)
        with open(tmp, "w") as f:
            f.write(key)
        os.replace(tmp, CALLS_KEY)
    finally:
        if os.path.exists(tmp):
            os.remove(tmp)
    return CALLS


def build(verbose: bool = False, extra=(), calls: bool = True) -> str:
    """Every source to an object file of its own (in parallel; no device code crosses a file), then one link.  calls: the
    extension module too; where that fails the library is in place all the same."""
    from concurrent.futures import ThreadPoolExecutor

    os.makedirs(OBJ, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]
    objs = []
    jobs = []
    for src in sources():
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        jobs.append(["hipcc", *compile_flags, *extra, "-c", src, "-o", obj])
    with ThreadPoolExecutor(max_workers=min(8, len(jobs))) as pool:
        module = pool.submit(build_calls, verbose) if calls else None
        list(pool.map(lambda cmd: _run(cmd, verbose), jobs))
        _run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB], verbose)
        if module:
            module.result()
    return LIB


if __name__ == "__main__":
    print(build(verbose=True, extra=sys.argv[1:]))
