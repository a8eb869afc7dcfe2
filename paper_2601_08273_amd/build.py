"""Build the HIP library and its binding in-tree: ``python -m paper_2601_08273_amd.build``.

hipcc cross-compiles for gfx950 without a GPU.  The results, ``libhippo.so`` and ``_binding.so`` (the entry points'
marshalling, host code against torch's headers), sit next to this file so that they travel with the source tree; they
are not installed anywhere.
"""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libhippo.so")
BINDING = os.path.join(HERE, "_binding.so")
SOURCES = ["api.hip", "attention.hip", "quantize.hip", "score.hip", "select_gather.hip", "spec_verify.hip", "vpsd.cpp"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 instruction forms
    "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def _compile(src: str, extra) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = ["hipcc", *FLAGS, *extra, *(["-x", "hip"] if src.endswith(".cpp") else []), "-c", os.path.join(CSRC, src),
           "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in r.stdout.splitlines() if "not a recognized feature" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    if out.strip():
        print(out)
    return obj


def _build_binding() -> None:
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = BINDING + ".tmp%d" % os.getpid()
    subprocess.check_call([
        "g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM",
        "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I", os.path.join(ROOT, "include"),
        "-isystem", os.path.join(root, "include"), "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
        "-isystem", "/opt/rocm/include", "-isystem", sysconfig.get_paths()["include"],
        os.path.join(CSRC, "binding.cpp"), "-o", tmp, "-L", os.path.join(root, "lib"),
        "-ltorch_python", "-ltorch_cpu", "-lc10", "-lc10_hip", "-ldl"])
    os.replace(tmp, BINDING)


def build(extra_flags=(), verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with ThreadPoolExecutor(max_workers=4) as ex:
        binding = ex.submit(_build_binding)
        objs = list(ex.map(lambda s: _compile(s, list(extra_flags)), SOURCES))
        binding.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp, *objs])
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB, BINDING)
    return LIB


if __name__ == "__main__":
    build(sys.argv[1:])
