"""Build libmamba_hip.so (gfx950, hipcc) and the binding's marshalling module (host C++) in-tree.
Usage: python -m paper_2506_01206_amd.build"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJDIR = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libmamba_hip.so")
MARSHAL = os.path.join(HERE, "_marshal.so")
SOURCES = ["api.cpp", "sd_tree_search.cpp", "conv1d.hip", "scan.hip", "scan_direct.hip", "scan_lanes.hip", "strided.hip", "step.hip", "fork.hip", "linear.hip", "draft_in.hip", "xdt.hip", "norm.hip", "vocab.hip", "ssd.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
# packed-fp32 VALU instructions are switched off for every device function.  The first 14 dwords of a kernel's arguments, up to
# the first aggregate, come in registers instead of through a scalar load (a trip to the cache that every address waits for).
# us of a launch in a chain, without / with: 12 x 768 product of k = 1536 3.32 / 3.10, fused layer step 32 x 1536 3.92 / 3.47, RMSNorm of 8000
# rows 7.65 / 7.24, scalar-decay scan of 1000 tokens 30.5 / 30.0.  Three kernels that do little but wait for memory lose
# by it (scalar-decay step of 4 branches 3.52 / 3.91, state step 1 x 768 1.95 / 2.04, embedding of 12 tokens 1.81 / 1.95): their
# first argument is an aggregate.
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-x", "hip",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=16", "-Wall", "-Wno-unused-function"]


def _compile(src: str) -> str:
    obj = os.path.join(OBJDIR, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    msgs = "\n".join(l for l in (r.stdout + r.stderr).splitlines()
                     if "packed-fp32-ops" not in l and "unknown target" not in l.lower())
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, r.stdout + r.stderr))
    if msgs.strip():
        sys.stderr.write(msgs + "\n")
    return obj


def marshal_command(out: str, compiler: str, flags=("-O2", "-Wall")) -> list:
    """How the native half of binding.py is compiled: host code against torch's C++ headers (device memory and streams only)."""
    import torch
    root = os.path.dirname(torch.__file__)
    return ([compiler, *flags, "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI]
            + ["-isystem" + d for d in (os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
                                        sysconfig.get_paths()["include"], os.path.join(os.path.dirname(os.path.dirname(HIPCC)), "include"))]
            + [os.path.join(CSRC, "marshal.cpp"), "-o", out, "-L" + os.path.join(root, "lib")]
            + ["-l" + n for n in ("torch_python", "torch_cpu", "torch", "c10", "c10_hip")])


def _build_marshal() -> None:
    tmp = MARSHAL + ".tmp%d" % os.getpid()
    subprocess.check_call(marshal_command(tmp, os.environ.get("CXX", "g++")))
    os.replace(tmp, MARSHAL)


def build(verbose: bool = False) -> str:
    """Compile every source, link libmamba_hip.so next to this file, and build the marshalling module."""
    os.makedirs(OBJDIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        marshal = ex.submit(_build_marshal)
        objs = list(ex.map(_compile, SOURCES))
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    marshal.result()
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
