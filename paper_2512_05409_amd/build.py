"""Builds libsq.so (the HIP kernels and their C ABI) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import glob
import hashlib
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libsq.so")

SOURCES = ["sq_encode.hip", "sq_encode_dyn.hip", "sq_encode_few.hip", "sq_encode_static.hip", "sq_storage.hip", "sq_wsq.hip", "sq_gemm.hip", "sq_gemm_few.hip", "sq_probe.hip", "sq_calib.hip", "sq_noalloc.hip", "sq_api.cpp"]

# -ffp-contract=off: the encoder's multiply-then-round and the epilogue's multiply / fma / multiply
# must stay the separate fp32 operations the layer is defined with.
# packed-fp32-ops are switched off for the device code on purpose.
HIP_FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-ffp-contract=off", "-fno-fast-math",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wall", "-Wno-unused-function",
             "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.sep not in c or os.path.exists(c)):
            return c
    raise RuntimeError("hipcc not found")


def sources_digest() -> str:
    """Digest of everything the library is compiled from: the sources, the headers and the flags."""
    h = hashlib.sha256(" ".join(f for f in HIP_FLAGS if not f.startswith("-I")).encode())
    files = [os.path.join(CSRC, s) for s in sorted(SOURCES)] + sorted(glob.glob(os.path.join(CSRC, "*.h")))
    for path in files + [os.path.join(ROOT, "include", "sq.h")]:
        with open(path, "rb") as f:
            h.update(os.path.basename(path).encode() + b"\0" + f.read() + b"\0")
    return h.hexdigest()


def _compile(src: str, digest: str) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [_hipcc()] + HIP_FLAGS + [f'-DSQ_SOURCES="{digest}"', "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("hipcc failed on " + src)
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and "unused during compilation" not in l)
    if warn.strip():
        sys.stderr.write(warn + "\n")
    return obj


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    digest = sources_digest()
    with ThreadPoolExecutor(max_workers=4) as ex:
        objs = list(ex.map(_compile, SOURCES, [digest] * len(SOURCES)))
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError("link failed")
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
