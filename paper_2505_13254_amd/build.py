"""Builds libheterospec.so (HIP, gfx950) in-tree with hipcc.  `python -m paper_2505_13254_amd.build`."""
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


def build(verbose: bool = True) -> str:
    """Compiles every source and links the shared library, and the binding's native module; always rebuilds."""
    objdir = os.path.join(PKG, "_build")
    os.makedirs(objdir, exist_ok=True)
    objs = []
    procs = []
    cmd = marshal_command()
    if verbose:
        print(" ".join(cmd), flush=True)
    procs.append(("marshal.cpp", subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [hipcc()] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        procs.append((src, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
        objs.append(obj)
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError("compiling %s failed:\n%s" % (src, out))
        if verbose and out.strip():
            print(out)
    cmd = [hipcc(), "-shared", "-fPIC", "--offload-arch=gfx950", "-o", LIB] + objs
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    return LIB


if __name__ == "__main__":
    build()
    print("built", LIB)
    sys.exit(0)
