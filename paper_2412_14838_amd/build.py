"""Builds libdkv.so (HIP kernels + C ABI) for gfx950, in-tree, with hipcc.

Usage: python -m paper_2412_14838_amd.build
"""
from __future__ import annotations

import concurrent.futures as cf
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libdkv.so")
BINDING = os.path.join(HERE, "_binding.so")

# packed fp32 VALU forms are switched off for all device code
HIPCC_FLAGS = ["-O3", "-fno-honor-nans", "-std=c++17", "--offload-arch=gfx950", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-Wall", "-Wno-unused-function"]
# An option of the compiler's code generator: results of matrix instructions in vector registers, where the exponentials read them. Without it
# a kernel of more than 256 registers has them in accumulation registers and copies them from there (16 instructions a unit of 8 products).
# For speed only. The kernels that it changes, us without / with it: the second sweep of 129 to 256 rows (28 layers of 4 heads x 32768 keys,
# 160, 192, 224, 256 rows 245 / 230, 275 / 260, 303 / 286, 342 / 310) and the first sweep of up to 64 rows (both sweeps: one layer of 8 heads,
# 2048 keys 12.0 / 11.6, 16384 keys 15.6 / 14.7, 64 prompts of 300 keys 30.4 / 28.8, 8 layers of 16 prompts of 1000 144 / 136; 32 layers
# of 32768 707 to 720 / 710 to 713, the same).
SOURCE_FLAGS = {"score_mfma.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = ["hipcc", *HIPCC_FLAGS, *SOURCE_FLAGS.get(os.path.basename(src), []), "-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
    noise = "'-packed-fp32-ops' is not a recognized feature"
    err = "\n".join(l for l in r.stderr.splitlines() if noise not in l)
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def build(verbose: bool = True) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    with cf.ThreadPoolExecutor(max_workers=min(8, len(srcs))) as ex:
        objs = list(ex.map(_compile, srcs))
    # Link against the HIP runtime that PyTorch loads (its own libamdhip64.so, found by name), not a second
    # copy: streams and graph captures created by torch are then valid inside the library.
    import torch
    torch_lib = os.path.join(os.path.dirname(torch.__file__), "lib")
    cmd = ["g++", "-shared", "-fPIC", "-o", LIB, *objs, "-L" + torch_lib, "-lamdhip64",
           "-Wl,-rpath," + torch_lib, "-Wl,-rpath,/opt/rocm/lib"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("link failed:\n%s\n%s" % (r.stdout, r.stderr))
    # the Python binding of the stage calls (host code only), beside the library and linked to it
    cmd = ["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-Wall", "-I" + sysconfig.get_paths()["include"], "-o", BINDING,
           os.path.join(CSRC, "binding.cpp"), "-L" + HERE, "-l:libdkv.so", "-Wl,-rpath,$ORIGIN"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("g++ failed for binding.cpp:\n%s\n%s" % (r.stdout, r.stderr))
    if verbose:
        print("built", LIB)
    # the stand-alone measurement programs under tests/probes (not part of the library)
    probes = os.path.join(os.path.dirname(HERE), "tests", "probes")
    for src in sorted(glob.glob(os.path.join(probes, "*.hip"))):
        exe = src[:-4]
        r = subprocess.run(["hipcc", "-O3", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                            "-o", exe, src], capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s\n%s" % (src, r.stdout, r.stderr))
        if verbose:
            print("built", exe)
    return LIB


if __name__ == "__main__":
    build()
