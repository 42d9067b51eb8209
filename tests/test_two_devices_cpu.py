"""A process that uses a second GPU: what a kernel has to be given on each device (more than 64 KB of dynamic LDS, asked for
with hipFuncSetAttribute) is asked for on each. The HIP calls of the library go to stand-ins that record them; nothing is
launched, no GPU is needed."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_INS = r"""
#include <stddef.h>
struct d3 { unsigned x, y, z; };
static int device, calls[64];
static const void* asked[64][256];
static struct { d3 grid, block; size_t lds; void* stream; } config;
extern "C" {
int stand_in_set_device(int d) { return device = d; }
int stand_in_calls(int d) { return calls[d]; }
const void* stand_in_kernel(int d, int i) { return asked[d][i]; }
int hipGetDevice(int* d) { *d = device; return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }
int hipFuncSetAttribute(const void* f, int, int) { asked[device][calls[device]++ % 256] = f; return 0; }
int hipGetLastError() { return 0; }
int hipLaunchKernel(const void*, d3, d3, void**, size_t, void*) { return 0; }
int __hipPushCallConfiguration(d3 grid, d3 block, size_t lds, void* stream) { config = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(d3* grid, d3* block, size_t* lds, void** stream) {
  *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
  return 0;
}
}
"""

PROGRAM = r"""
import ctypes as C, json, sys
stand_ins = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
stand_ins.stand_in_kernel.restype = C.c_void_p
from paper_2412_14838_amd import dkv
lib = C.CDLL(dkv.LIB_PATH)
P, I64 = C.c_void_p, C.c_int64
fake, big = P(0x10000), C.c_size_t(1 << 50)
found = []
for dtype, d in ((dkv.DKV_F32, 64), (dkv.DKV_F32, 128), (dkv.DKV_BF16, 64), (dkv.DKV_BF16, 128)):
    desc = dkv.make_desc(n_layers=2, n_q_heads=8, n_kv_heads=2, head_dim=d, window=16, pool_kernel=7, layer_max=64,
                         mean_budget=32, interval=1, dtype=dtype, n_seqs=1, total_tokens=1024, max_seq_len=1024)
    for device in (0, 5, 0, 5):
        stand_ins.stand_in_set_device(device)
        before = stand_ins.stand_in_calls(device)
        assert lib.dkv_score_window(C.byref(desc), fake, fake, I64(d), I64(1024 * d), fake, fake, I64(1024), fake, big, None) == 0
        assert lib.dkv_select_topk(C.byref(desc), 0, fake, I64(1024), fake, fake, fake, fake, big, None) == 0
        kernels = sorted({stand_ins.stand_in_kernel(device, i) for i in range(before, stand_ins.stand_in_calls(device))})
        found.append([dtype, d, device, kernels])
print(json.dumps(found))
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_dynamic_lds_is_asked_for_on_every_device(tmp_path):
    src, lib = tmp_path / "stand_ins.cpp", tmp_path / "libstand_ins.so"
    src.write_text(STAND_INS)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    run = subprocess.run([sys.executable, "-c", PROGRAM, str(lib)], capture_output=True, text=True, cwd=ROOT, timeout=300)
    assert run.returncode == 0, run.stderr
    found = json.loads(run.stdout.strip().splitlines()[-1])
    for i in range(0, len(found), 4):
        first, second, again, second_again = (x[3] for x in found[i:i + 4])
        assert first and second == first, found[i]               # the same kernels on both
        assert again == [] and second_again == []                # and once


UNITS_STAND_INS = STAND_INS.replace("int hipDeviceGetAttribute(int* v, int, int) { *v = 256; return 0; }",
                                    "int hipDeviceGetAttribute(int* v, int, int d) { *v = d == 5 ? 24 : 256; return 0; }").replace(
    "int hipLaunchKernel(const void*, d3, d3, void**, size_t, void*) { return 0; }",
    "static int launches; int stand_in_launches() { return launches; }\n"
    "int hipLaunchKernel(const void*, d3, d3, void**, size_t, void*) { ++launches; return 0; }")

UNITS_PROGRAM = r"""
import ctypes as C, json, sys
stand_ins = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2412_14838_amd import dkv
lib = C.CDLL(dkv.LIB_PATH)
P, I64 = C.c_void_p, C.c_int64
fake, big = P(0x10000), C.c_size_t(1 << 50)
desc = dkv.make_desc(n_layers=2, n_q_heads=32, n_kv_heads=8, head_dim=128, window=16, pool_kernel=7, layer_max=64, mean_budget=32,
                     interval=1, dtype=dkv.DKV_BF16, n_seqs=1, total_tokens=1024, max_seq_len=1024)
found = []
for device in json.loads(sys.argv[2]):
    stand_ins.stand_in_set_device(device)
    before = stand_ins.stand_in_launches()
    assert lib.dkv_decode_attention(C.byref(desc), 0, fake, fake, fake, I64(8 * 80 * 128), I64(80 * 128), fake, fake, fake, fake, fake,
                                    big, None) == 0
    found.append(stand_ins.stand_in_launches() - before)
print(json.dumps(found))
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("devices", [[0, 5, 0, 5], [5, 0, 5, 0]])
def test_every_device_is_asked_for_its_compute_units(tmp_path, devices):
    """A call of 32 workgroups fits 256 compute units at once (one kernel) and 24 not (two), whichever device came first."""
    src, lib = tmp_path / "stand_ins.cpp", tmp_path / "libstand_ins.so"
    src.write_text(UNITS_STAND_INS)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    run = subprocess.run([sys.executable, "-c", UNITS_PROGRAM, str(lib), json.dumps(devices)], capture_output=True, text=True, cwd=ROOT,
                         timeout=300)
    assert run.returncode == 0, run.stderr
    assert json.loads(run.stdout.strip().splitlines()[-1]) == [2 if d == 5 else 1 for d in devices]
