"""Builds libtokenring.so (HIP, gfx950 only) in-tree with hipcc.

The library carries a hash of everything it was compiled from (kernel sources, internal and
public headers, compiler flags): tr_version() reports it, and ensure_built() recompiles when
the hash found inside an existing library differs from the hash of the sources on disk, so a
test or benchmark run can never silently exercise a stale binary.  The hash in the Python module over it
covers torch's version and C++ ABI and Python's, which it is compiled against, as well.
"""
from __future__ import annotations

import hashlib
import os
import re
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG_DIR)
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB_PATH = os.path.join(PKG_DIR, "libtokenring.so")
BINDING_PATH = os.path.join(PKG_DIR, "_native.so")   # Python module over it
SOURCES = ["api.hip", "merge.hip", "block_attn.hip"] + [f"block_attn_d{d}_{r}rows.hip" for d in (128, 64) for r in (256, 128, 64)]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    # packed-fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]
CXX_FLAGS = ["-O2", "-std=c++17", "-fPIC", "-Wall"]
_HASH_TAG = b"TR_SOURCE_HASH="


def source_hash() -> str:
    """Hex digest (16 characters) over every file of csrc/ and include/ plus the compiler flags."""
    h = hashlib.sha256()
    h.update(" ".join(HIPCC_FLAGS).encode())
    for folder in (CSRC, INCLUDE):
        for name in sorted(os.listdir(folder)):
            path = os.path.join(folder, name)
            if os.path.isfile(path) and name.endswith((".hip", ".cpp", ".h", ".hpp", ".inc")):
                h.update(name.encode() + b"\0")
                with open(path, "rb") as f:
                    h.update(f.read())
                h.update(b"\0")
    return h.hexdigest()[:16]


def binding_hash() -> str:
    """The same for the Python module: the sources, its compiler's flags, and the torch and Python it is compiled against."""
    import torch
    what = [source_hash(), *CXX_FLAGS, torch.__version__, str(torch._C._GLIBCXX_USE_CXX11_ABI), sysconfig.get_config_var("SOABI") or sys.version]
    return hashlib.sha256("\0".join(what).encode()).hexdigest()[:16]


def library_hash(path: str = LIB_PATH):
    """The source hash embedded in a built library (read from the file, nothing is loaded); None if absent."""
    if not os.path.exists(path):
        return None
    with open(path, "rb") as f:
        m = re.search(re.escape(_HASH_TAG) + rb"([0-9a-f]{16})", f.read())
    return m.group(1).decode() if m else None


def build_library(verbose: bool = False) -> str:
    """Compile every kernel source into one shared library, and the Python module over it; returns the library's path."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp, tmp_binding = LIB_PATH + f".tmp{os.getpid()}", BINDING_PATH + f".tmp{os.getpid()}"
    objects = [f"{tmp}.{s}.o" for s in SOURCES]
    compile_ = [hipcc, *HIPCC_FLAGS, f'-DTR_SOURCE_HASH_STR="{source_hash()}"', "-I", INCLUDE, "-I", CSRC, "-c"]

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        noise = "is not a recognized feature for this target"
        err = "\n".join(l for l in res.stderr.splitlines() if noise not in l)
        if res.returncode != 0:
            raise RuntimeError(f"{os.path.basename(cmd[0])} failed ({res.returncode}):\n{err}")
        if verbose and err.strip():
            print(err, file=sys.stderr)

    import torch   # its headers and libraries
    torch_root = os.path.dirname(torch.__file__)
    cxx, binding = os.environ.get("CXX", "g++"), tmp_binding + ".o"
    compile_binding = [cxx, *CXX_FLAGS, f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
                       f'-DTR_SOURCE_HASH_STR="{binding_hash()}"', "-I", INCLUDE, "-isystem", sysconfig.get_paths()["include"],
                       "-isystem", os.path.join(torch_root, "include"), "-c", os.path.join(CSRC, "binding.cpp"), "-o", binding]
    commands = [[*compile_, os.path.join(CSRC, s), "-o", o] for s, o in zip(SOURCES, objects)] + [compile_binding]
    try:
        with ThreadPoolExecutor(min(len(commands), os.cpu_count() or 1, 8)) as pool:   # one compiler per source
            for done in [pool.submit(run, cmd) for cmd in commands]:
                done.result()
        run([hipcc, *HIPCC_FLAGS, "-shared", "-o", tmp, *objects])
        os.replace(tmp, LIB_PATH)      # atomic: a concurrent reader never sees a half-written library
        run([cxx, "-shared", "-o", tmp_binding, binding, "-L", os.path.join(torch_root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
             "-L", PKG_DIR, "-l:" + os.path.basename(LIB_PATH), "-Wl,-rpath,$ORIGIN"])
        os.replace(tmp_binding, BINDING_PATH)
    finally:
        for o in (*objects, binding, tmp, tmp_binding):
            if os.path.exists(o):
                os.remove(o)
    return LIB_PATH


def ensure_built() -> str:
    """Build unless a library compiled from exactly the sources on disk is already there, and a module that fits this torch and Python."""
    if library_hash() == source_hash() and library_hash(BINDING_PATH) == binding_hash():
        return LIB_PATH
    return build_library()


if __name__ == "__main__":
    print(build_library(verbose="-v" in sys.argv))
