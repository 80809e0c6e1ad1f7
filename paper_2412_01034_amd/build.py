"""Builds libqail.so in-tree with hipcc for gfx950 (cross-compiles without a GPU)."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libqail.so")
MARSHAL = os.path.join(HERE, "_marshal" + sysconfig.get_config_var("EXT_SUFFIX"))   # another Python does not look at it

SOURCES = ("api.hip", "quantize.hip", "w4a16_gemv.hip", "w4a16_decode4.hip", "w4a16_smallm.hip", "w4a16_midm.hip", "w4a16_gemm.hip", "w4a16_generic.hip", "w4a16_lora.hip", "w8.hip", "w8a16_gemv.hip", "train_ops.hip", "w4a4_conv.hip")

HIPCC_FLAGS = (
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-Wall", "-Wno-unused-command-line-argument",
)


def _hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    return "hipcc"


def _run(cmd):
    p = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in p.stdout.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def build_marshal() -> str:
    """Compile the binding's marshalling (csrc/marshal.cpp) against this Python and this torch, whose names it keeps."""
    import torch
    top = os.path.dirname(torch.__file__)
    tmp = MARSHAL + ".tmp"
    _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-w", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
          '-DQAIL_TORCH="%s %s"' % (torch.__version__, torch.version.git_version), "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I", os.path.join(ROOT, "include"),
          "-I", sysconfig.get_paths()["include"], "-I", os.path.join(top, "include"),
          "-I", os.path.join(top, "include", "torch", "csrc", "api", "include"), "-I", "/opt/rocm/include",
          os.path.join(CSRC, "marshal.cpp"), "-o", tmp, "-L", os.path.join(top, "lib"),
          "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-lc10_hip"])
    os.replace(tmp, MARSHAL)
    return MARSHAL


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source and link libqail.so next to this file, and the binding's marshalling beside it.

    The library needs hipcc alone.  Without a host compiler or the headers of Python and torch there is no marshalling, and the
    binding does that work in Python."""
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    hipcc = _hipcc()

    def compile_one(src):
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        out = _run([hipcc, *HIPCC_FLAGS, *inc, "-c", os.path.join(CSRC, src), "-o", obj])
        if verbose and out.strip():
            print(out, file=sys.stderr)
        return obj

    for old in glob.glob(os.path.join(os.path.dirname(MARSHAL), "_marshal*.so")):   # what is not built anew is not used
        os.remove(old)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as ex:
        marshal = ex.submit(build_marshal)
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    _run([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if marshal.exception() is not None:
        print("calls are marshalled in Python, csrc/marshal.cpp was not built: %s" % marshal.exception(), file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
