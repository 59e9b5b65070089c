"""Builds libbastion_tv.so for gfx950 with hipcc (cross-compiles without a GPU), and _face.so, its face for torch, with g++."""
from __future__ import annotations

import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libbastion_tv.so")
FACE = os.path.join(HERE, "_face.so")
SOURCES = ["api.hip", "attn.hip", "tree_build.hip", "accept.hip", "lm_head.hip", "stochastic.hip", "kv_commit.hip"]

# -packed-fp32-ops is switched off: the compiler must not form packed fp32 VALU ops on this target.
# Kernel arguments that are scalars or pointers come in registers with a wavefront's start (the first 14 words of them) instead of by loads
# that the first instructions wait for: 0.2 to 0.7 us of a call (LM head, 16 nodes, h = 2560, V = 32000: 36.9 -> 36.1; h = 1024, V = 9000:
# 11.55 -> 11.36; tree build, 256 nodes 25.35 -> 25.0).
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-mllvm", "-amdgpu-kernarg-preload-count=16", "-I", INCLUDE, "-I", CSRC]


def _face_command() -> list:
    import sysconfig
    import torch
    from torch.utils import cpp_extension
    libs = cpp_extension.library_paths()
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
             f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", "-I", INCLUDE, "-I", sysconfig.get_paths()["include"]]
            + [x for p in cpp_extension.include_paths() + ["/opt/rocm/include"] for x in ("-isystem", p)]
            + [os.path.join(CSRC, "face.cpp"), "-o", FACE, "-L", HERE, "-l:libbastion_tv.so", "-Wl,-rpath,$ORIGIN"]
            + [x for p in libs for x in ("-L", p)] + ["-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip"])


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs = []
    procs = []
    os.makedirs(os.path.join(HERE, "_build"), exist_ok=True)
    for src in SOURCES:
        obj = os.path.join(HERE, "_build", src.replace(".hip", ".o"))
        objs.append(obj)
        procs.append((src, subprocess.Popen([hipcc, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj],
                                            stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)))
    for src, p in procs:
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "packed-fp32-ops" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"hipcc failed on {src}:\n{out}")
        if verbose and out.strip():
            print(out)
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs])
    p = subprocess.run(_face_command(), stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if p.returncode != 0:
        raise RuntimeError(f"g++ failed on face.cpp:\n{p.stdout}")
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
