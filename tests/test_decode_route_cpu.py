"""Which kernels a decode call takes: one, or the two of larger calls. The HIP calls go to stand-ins that count launches: no GPU is
needed."""
import json
import shutil
import subprocess
import sys

import pytest

from paper_2412_14838_amd import dkv
from test_two_devices_cpu import ROOT, UNITS_STAND_INS

PROGRAM = r"""
import ctypes as C, json, sys
stand_ins = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
from paper_2412_14838_amd import dkv
lib = C.CDLL(dkv.LIB_PATH)
P, I64 = C.c_void_p, C.c_int64
fake, big = P(0x10000), C.c_size_t(1 << 50)
found = []
for Hkv, G, d, w, mean, layer_max, n_seqs, dtype in json.loads(sys.argv[2]):
    desc = dkv.make_desc(n_layers=2, n_q_heads=Hkv * G, n_kv_heads=Hkv, head_dim=d, window=w, pool_kernel=7, layer_max=layer_max,
                         mean_budget=mean, interval=1, dtype=dtype, n_seqs=n_seqs, total_tokens=4096, max_seq_len=4096)
    before, block = stand_ins.stand_in_launches(), (w + layer_max) * d
    assert lib.dkv_decode_attention(C.byref(desc), 0, fake, fake, fake, I64(Hkv * block), I64(block), fake, fake, fake, fake, fake, big,
                                    None) == 0
    found.append(stand_ins.stand_in_launches() - before)
print(json.dumps(found))
"""
BF16, F32 = dkv.DKV_BF16, dkv.DKV_F32
CASES = [                                                    # Hkv, G, d, w, mean budget, layer_max, sequences, type: launches
    ((8, 4, 128, 32, 608, 2048, 1, BF16), 1), ((8, 4, 128, 32, 609, 2048, 1, BF16), 2),      # rows to expect: 640, 641
    ((8, 4, 128, 32, 2048, 2048, 1, BF16), 2), ((8, 4, 128, 32, 2048, 608, 1, BF16), 1),     # never more than layer_max
    ((8, 4, 128, 32, 2 ** 31 - 1, 2048, 1, BF16), 2), ((8, 4, 128, 32, 2 ** 31 - 1, 600, 1, BF16), 1),
    ((8, 4, 128, 32, 128, 512, 8, BF16), 1), ((8, 4, 128, 32, 128, 512, 9, BF16), 2),        # workgroups: 256, 288 of 256
    ((8, 4, 64, 32, 128, 512, 16, BF16), 1), ((8, 4, 64, 32, 128, 512, 17, BF16), 2),
    ((8, 16, 128, 16, 128, 1136, 1, BF16), 1), ((8, 16, 128, 16, 128, 1137, 1, BF16), 2),    # LDS: 9, 10 slabs of 16 heads
    ((8, 4, 128, 32, 128, 512, 1, F32), 2),
]


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_route_of_a_call(tmp_path):
    src, lib = tmp_path / "stand_ins.cpp", tmp_path / "libstand_ins.so"
    src.write_text(UNITS_STAND_INS)
    subprocess.run(["g++", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    run = subprocess.run([sys.executable, "-c", PROGRAM, str(lib), json.dumps([c for c, _ in CASES])], capture_output=True, text=True,
                         cwd=ROOT, timeout=300)
    assert run.returncode == 0, run.stderr
    assert list(zip([c for c, _ in CASES], json.loads(run.stdout.strip().splitlines()[-1]))) == CASES
