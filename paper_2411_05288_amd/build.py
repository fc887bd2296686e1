"""Builds libvp.so (the C-ABI library with the HIP kernels) for gfx950 with hipcc, and _vphost.so, the tensor checks of the
Python binding, with the host compiler against PyTorch's headers.

Usage:  python -m paper_2411_05288_amd.build
The library is placed next to this file so that it travels with the source tree.
"""
from __future__ import annotations

import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libvp.so")
HOST = os.path.join(HERE, "_vphost.so")
OBJDIR = os.path.join(HERE, "_build")

SOURCES = ["vp_api.hip", "vp_profile.hip", "vp_gemm_bf16.hip", "vp_gemm_bf16_logits.hip", "vp_gemm_bf16_fast.hip", "vp_gemm_bf16_twin.hip", "vp_gemm_f32.hip", "vp_stats.hip", "vp_embed.hip"]

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
    # keep the compiler from forming packed fp32 VALU ops
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _run(cmd):
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("command failed: %s\n%s" % (" ".join(cmd), out))
    return out


def _host():
    import sysconfig

    import torch
    root = os.path.dirname(torch.__file__)
    rocm = os.path.dirname(os.path.dirname(HIPCC))
    tmp = HOST + ".tmp"
    out = _run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1",
                "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
                *["-isystem" + d for d in (os.path.join(root, "include"),
                                           os.path.join(root, "include", "torch", "csrc", "api", "include"),
                                           sysconfig.get_paths()["include"], os.path.join(rocm, "include"))],
                os.path.join(CSRC, "vp_host.cpp"), "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
                "-lc10_hip", "-o", tmp])
    os.replace(tmp, HOST)
    return out


def build(verbose: bool = False) -> str:
    os.makedirs(OBJDIR, exist_ok=True)
    objs = [os.path.join(OBJDIR, s.replace(".hip", ".o")) for s in SOURCES]

    def one(i):
        return _run([HIPCC, *FLAGS, "-c", os.path.join(CSRC, SOURCES[i]), "-o", objs[i]])

    with ThreadPoolExecutor(max_workers=8) as ex:
        host = ex.submit(_host)
        for out in ex.map(one, range(len(SOURCES))):
            if verbose and out.strip():
                print(out)
        host.result()
    tmp = LIB + ".tmp"
    _run([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
    sys.exit(0)
