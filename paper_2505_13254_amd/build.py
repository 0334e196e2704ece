"""Builds libheterospec.so (HIP, gfx950) in-tree with hipcc, and the binding's native module.  `python -m
paper_2505_13254_amd.build`; the library alone, without torch: `python paper_2505_13254_amd/build.py --library`."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libheterospec.so")
MARSHAL = os.path.join(PKG, "_marshal.so")  # host only: Python tensors -> the library's calls (csrc/marshal.cpp)
SOURCES = ["api.cpp", "entropy_topk.hip", "tree_prune.hip", "tree_attention.hip", "tree_attention_mfma.hip",
           "verify_accept.hip", "tree_expand.hip", "adaptive_control.hip", "kv_commit.hip", "tree_validate.hip"]
FLAGS = ["-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950", "-x", "hip",
         # packed-fp32 instruction selection is switched off for every device function of the library
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-Wall", "-Wno-unused-variable"]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found")
    return exe


def marshal_command():
    """The host compiler's line for the binding's native module, against the torch that is installed."""
    import sysconfig

    import torch
    t = os.path.dirname(torch.__file__)
    return [shutil.which("g++") or "c++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
            "-I" + os.path.join(ROOT, "include"), "-isystem", sysconfig.get_paths()["include"],
            "-isystem", os.path.join(t, "include"), "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
            os.path.join(CSRC, "marshal.cpp"), "-L" + os.path.join(t, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10", "-o", MARSHAL]


def _start(cmd, verbose: bool):
    if verbose:
        print(" ".join(cmd), flush=True)
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _finish(src: str, p, verbose: bool) -> None:
    out, _ = p.communicate()
    out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
    if p.returncode != 0:
        raise RuntimeError("compiling %s failed:\n%s" % (src, out))
    if verbose and out.strip():
        print(out)


def build_library(verbose: bool = True) -> str:
    """Compiles every source and links the shared library, with hipcc and nothing else; always rebuilds."""
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = [os.path.join(objdir, os.path.splitext(src)[0] + ".o") for src in SOURCES]
    procs = [(src, _start([hipcc()] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj], verbose)) for src, obj in zip(SOURCES, objs)]
    for src, p in procs:
        _finish(src, p, verbose)
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


def build(verbose: bool = True) -> str:
    """The shared library, and the binding's native module beside it, which needs torch, Python's headers and a host
    compiler: where that fails, the library is there all the same when the error is raised."""
    marshal, failed = None, None
    try:
        marshal = _start(marshal_command(), verbose)
    except Exception as e:
        failed = e
    build_library(verbose)
    if marshal is None:
        raise RuntimeError("the binding's native module was not compiled (the library was)") from failed
    _finish("marshal.cpp", marshal, verbose)
    return LIB


if __name__ == "__main__":  # --library: libheterospec.so alone, for users of the C interface
    if "--library" in sys.argv[1:]:
        build_library()
    else:
        build()
    print("built", LIB)
    sys.exit(0)
