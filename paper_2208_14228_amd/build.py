"""Builds libes.so (HIP, gfx950 only) in-tree with hipcc."""
from __future__ import annotations

import hashlib
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libes.so")
STAMP = LIB + ".srchash"
SOURCES = [os.path.join(CSRC, "es_kernels.hip"), os.path.join(CSRC, "es_api.cpp"),
           os.path.join(CSRC, "es_sched.cpp")]
HEADERS = [os.path.join(CSRC, "es_internal.h"), os.path.join(ROOT, "include", "es.h"),
           os.path.join(ROOT, "include", "es_sched.h")]

# The binding's native calls: an extension module of the running interpreter, where its headers are installed
# (without it the binding makes every call through ctypes).
PYCALL_SOURCE = os.path.join(CSRC, "es_pycall.cpp")
PYCALL = os.path.join(HERE, "_pycall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))
PYCALL_STAMP = os.path.join(HERE, "_pycall.srchash")

# -ffp-contract=off: no fused multiply-add may be formed (bit-exact SGD update)
# -fhip-fp32-correctly-rounded-divide-sqrt: IEEE division for the /N
# -fno-gpu-flush-denormals-to-zero: fp32 denormals are kept
# packed-fp32 instructions are switched off for the device code
# kernel arguments that are single words arrive in registers (as many as 16 hold) instead of by a load, whose round
# trip precedes every address of a short kernel
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero", "-fno-fast-math",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-kernarg-preload-count=16",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    return "hipcc"


def source_hash() -> str:
    """Identifies what a library was built from: the sources, the headers and the flags."""
    h = hashlib.sha256(" ".join(f for f in FLAGS if not os.path.isabs(f)).encode())
    for f in SOURCES + HEADERS:
        with open(f, "rb") as fh:
            h.update(os.path.basename(f).encode() + b"\0" + fh.read())
    return h.hexdigest()[:16]


def stale() -> bool:
    """True if there is no built library, or it was built from other sources than the tree holds
    (the hash of what it was built from sits beside it and is compiled into es_version())."""
    try:
        with open(STAMP) as fh:
            return not os.path.exists(LIB) or fh.read().strip() != source_hash()
    except OSError:
        return True


def pycall_hash() -> str:
    """Identifies what the extension module was built from and for; compiled into it as SOURCE_HASH."""
    h = hashlib.sha256(os.path.basename(PYCALL).encode())
    for f in (PYCALL_SOURCE, os.path.join(ROOT, "include", "es.h")):
        with open(f, "rb") as fh:
            h.update(b"\0" + fh.read())
    return h.hexdigest()[:16]


def build_pycall(force: bool, verbose: bool) -> None:
    include = sysconfig.get_paths()["include"]
    if not os.path.exists(os.path.join(include, "Python.h")):
        return
    tag = pycall_hash()
    if not force and os.path.exists(PYCALL):
        try:
            with open(PYCALL_STAMP) as fh:
                if fh.read().strip() == tag:
                    return
        except OSError:
            pass
    # (-x c++: hipcc takes it for an ordinary C++ file, no device code)
    cmd = [hipcc(), "-x", "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", include, "-I", os.path.join(ROOT, "include"),
           f'-DES_PYCALL_HASH="{tag}"', PYCALL_SOURCE, "-o", PYCALL]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    with open(PYCALL_STAMP, "w") as fh:
        fh.write(tag + "\n")


def build(force: bool = True, verbose: bool = False) -> str:
    if force or stale():
        tag = source_hash()
        cmd = [hipcc(), *FLAGS, f'-DES_SOURCE_HASH="{tag}"', *SOURCES, "-o", LIB]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)
        with open(STAMP, "w") as fh:
            fh.write(tag + "\n")
    build_pycall(force, verbose)
    return LIB


if __name__ == "__main__":
    print(build(force=True, verbose=True))
