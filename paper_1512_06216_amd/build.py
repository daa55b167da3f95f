"""Builds libpsd.so (the C-ABI HIP library, gfx950, hipcc) and _psdpy.so (the Python binding's native half, g++), in-tree."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libpsd.so")
EXT = os.path.join(PKG, "_psdpy.so")
SOURCES = ["psd_host.hip", "psd_dense.hip", "psd_pack.hip", "psd_sfb_f32.hip", "psd_sfb_planes.hip", "psd_sfb_bf16.hip", "psd_sfb_small.hip", "psd_bias.hip", "psd_static.hip", "psd_ssp.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-I", os.path.join(ROOT, "include"),
         "-I", CSRC, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def _compile(src):
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass does not know the packed-fp32 feature and says so: not an error
    out = "\n".join(l for l in r.stdout.splitlines() if "packed-fp32-ops" not in l)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s" % (src, out))
    return obj, out


def _torch_dir():
    import torch
    return os.path.dirname(os.path.abspath(torch.__file__))


def _compile_binding():
    """Host code only: the HIP headers are included for torch's stream type."""
    obj = os.path.join(OBJ, "psd_py.o")
    inc = os.path.join(_torch_dir(), "include")
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-I", os.path.join(ROOT, "include"),
           "-isystem", inc, "-isystem", os.path.join(inc, "torch", "csrc", "api", "include"), "-isystem", "/opt/rocm/include",
           "-I", sysconfig.get_paths()["include"], "-c", os.path.join(CSRC, "psd_py.cpp"), "-o", obj]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for psd_py.cpp:\n%s" % r.stdout)
    return obj


def build_library(verbose=False, jobs=None):
    os.makedirs(OBJ, exist_ok=True)
    jobs = jobs or min(len(SOURCES) + 1, max(1, (os.cpu_count() or 2) // 2))
    with ThreadPoolExecutor(jobs) as ex:
        binding_obj = ex.submit(_compile_binding)
        res = list(ex.map(_compile, SOURCES))
        binding_obj = binding_obj.result()
    for obj, out in res:
        if out.strip() and verbose:
            print(out, file=sys.stderr)
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *[o for o, _ in res]]
    subprocess.check_call(cmd)
    subprocess.check_call(["g++", "-shared", "-o", EXT, binding_obj, "-L", os.path.join(_torch_dir(), "lib"), "-ltorch_python", "-ltorch_cpu",
                           "-lc10", "-lc10_hip", "-L", PKG, "-lpsd", "-Wl,-rpath,$ORIGIN"])
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
