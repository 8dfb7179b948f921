"""Build step of the HIP library ``liblsefit.so`` (gfx950 only).

Compiles every ``csrc/*.hip`` translation unit with hipcc in parallel and links
them into ``paper_1512_08017_amd/liblsefit.so``.  Flags:

* ``--offload-arch=gfx950``                 MI355X (CDNA4) code objects only
* ``-O3 -std=c++20``
* ``-ffp-contract=off``                     no implicit FMA contraction; fused
                                             multiply-adds are written out
                                             explicitly where wanted, so the
                                             compensated sums keep their meaning
* ``-Xclang -target-feature -Xclang -packed-fp32-ops``
                                             no packed FP32 instructions

and ``csrc/bind.cpp`` (host code: the Python surface's argument marshalling)
with g++ into ``paper_1512_08017_amd/_bind.so``.
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "liblsefit.so")
OBJDIR = os.path.join(ROOT, "_build", "obj")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
CFLAGS = ["--offload-arch=" + ARCH, "-O3", "-std=c++20", "-fPIC", "-ffp-contract=off",
          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
          "-Wall", "-Wno-unused-function", "-I" + INCLUDE, "-I" + CSRC]


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(OBJDIR, os.path.basename(src) + ".o")
    cmd = [HIPCC, *CFLAGS, "-c", src, "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(line for line in res.stderr.splitlines() if "packed-fp32-ops" not in line)
    if res.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{err}")
    if err.strip() and verbose:
        print(err, file=sys.stderr)
    return obj


BIND = os.path.join(HERE, "_bind.so")


def build_bind(verbose: bool = False) -> str:
    import torch
    top = os.path.dirname(torch.__file__)
    inc = [INCLUDE, sysconfig.get_paths()["include"], os.path.join(top, "include"),
           os.path.join(top, "include", "torch", "csrc", "api", "include"), "/opt/rocm/include"]
    lib = os.path.join(top, "lib")
    tmp = BIND + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", *["-I" + i for i in inc],
           os.path.join(CSRC, "bind.cpp"), "-o", tmp, "-L" + lib, "-lc10", "-lc10_hip", "-ltorch_cpu",
           "-ltorch_python", "-Wl,-rpath," + lib]
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"g++ failed on bind.cpp:\n{res.stderr}")
    os.replace(tmp, BIND)
    return BIND


def build(verbose: bool = False, jobs: int | None = None) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    # the widest degree units take longest: start them first
    srcs.sort(key=lambda s: -int(s.rsplit("_m", 1)[1].split(".")[0]) if "_m" in os.path.basename(s) else 0)
    jobs = jobs or min(len(srcs), os.cpu_count() or 4, 16)
    with cf.ThreadPoolExecutor(max_workers=jobs + 1) as ex:
        bind = ex.submit(build_bind, verbose)
        objs = list(ex.map(lambda s: _compile(s, verbose), srcs))
        bind.result()
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=" + ARCH, "-shared", "-fPIC", "-o", tmp, *objs]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
