"""Build libvqmi.so (the C-ABI library of hand-written gfx950 kernels) in-tree with hipcc, and _marshal (the native part
of the Python binding) with the host compiler.

hipcc cross-compiles for gfx950 without a GPU, so this runs on the CPU build host;
the resulting shared object travels with the source tree to the GPU machine.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libvqmi.so")
MARSHAL = os.path.join(PKG, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))   # (another Python does not load it)
SOURCES = ["api.hip", "dequant.hip", "gemv.hip", "gemv_packed.hip", "gemv_mfma.hip", "gemv_replica.hip", "gemv_lut.hip", "gemm.hip", "gemm_skinny.hip", "gemm_dense.hip", "gemm_tiles.hip", "attn.hip", "attn_channel.hip", "kv_quantize.hip", "reorder.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Wall", "-Wno-unused-function",
         # packed fp32 VALU forms are disabled for every kernel of this library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *extra, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    warn = "\n".join(l for l in r.stderr.splitlines() if "packed-fp32-ops" not in l and l.strip())
    if warn.strip():
        sys.stderr.write(warn + "\n")
    return obj


def _build_marshal() -> None:
    import torch

    from .binding import marshal_built_for
    base = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(shutil.which(HIPCC) or HIPCC)))   # (HIPCC may be a name on PATH, or a link)
    tmp = MARSHAL + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI), '-DVQ_BUILT_FOR="%s"' % marshal_built_for()[0],
           "-I", os.path.join(ROOT, "include"),
           *(f"-isystem{p}" for p in (os.path.join(base, "include"), os.path.join(base, "include", "torch", "csrc", "api", "include"),
                                      os.path.join(rocm, "include"), sysconfig.get_paths()["include"])),
           os.path.join(CSRC, "marshal.cpp"), "-o", tmp, "-L", os.path.join(base, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("%s failed for marshal.cpp:\n%s" % (cmd[0], r.stderr))
    os.replace(tmp, MARSHAL)


def _build_marshal_if_possible() -> None:
    """The library does not need it, and neither does the binding: where it cannot be built (no torch or its headers, no host
    compiler) that is said, and calls are marshalled by ctypes."""
    try:
        _build_marshal()
    except Exception as e:  # noqa: BLE001
        sys.stderr.write("the native part of the binding was not built: %s\n" % e)
        if os.path.exists(MARSHAL):
            os.remove(MARSHAL)      # (that of an earlier build)


def build(extra_flags=(), jobs: int = 7) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        marshal = ex.submit(_build_marshal_if_possible)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
        marshal.result()
    tmp = LIB + ".tmp.%d" % os.getpid()
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs], check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(sys.argv[1:]))
