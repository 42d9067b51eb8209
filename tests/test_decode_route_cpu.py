"""Which kernels a decode call takes (one, or the two of larger calls), and what the layer loop tells the library about the rows a
layer keeps. The HIP calls go to stand-ins that count launches, the stage calls to recorders: no GPU is needed."""
import json
import shutil
import subprocess
import sys

import pytest
import torch

from paper_2412_14838_amd import dkv, pipeline as P, workloads as W
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


def _compressor(monkeypatch, **kw):
    seen = []
    for name in ("score_window", "score_window_layers", "select_topk", "select_topk_layers", "gather_kv", "gather_kv_layers", "rebalance",
                 "rebalance_batch", "apply_budgets", "select_recent"):
        monkeypatch.setattr(dkv, "dkv_" + name, lambda *a, **k: None)
    monkeypatch.setattr(dkv, "dkv_decode_attention", lambda desc, *a: seen.append((desc.mean_budget, desc.softmax_scale)))
    monkeypatch.setattr(dkv, "dkv_decode_attention_layers", lambda desc, *a: seen.append((desc.mean_budget, desc.softmax_scale)))
    cfg = W.Workload("route", L=6, Hq=4, Hkv=2, d=64, seqlens=(300, 70), dtype="bf16", w=16, P=7, mean_budget=10, layer_max=64, interval=4,
                     seed=1)
    comp = P.Compressor(cfg, device="cpu", **kw)
    comp.desc.softmax_scale = 0.25                              # whatever the caller's descriptor says goes with every call
    t = torch.zeros(1)

    def expected():
        del seen[:]
        for l in range(6):
            comp.decode_attention(l, t, t)
        for l, n in ((0, 6), (0, 4), (4, 2), (3, 2)):
            comp.decode_attention_layers(l, n, t, t)
        assert {s for _, s in seen} == {0.25} and comp.desc.mean_budget == 10
        return [r for r, _ in seen]

    return comp, t, expected


@pytest.mark.parametrize("group", [1, 4])
def test_layers_no_update_has_cut_are_said_to_hold_all_candidates(monkeypatch, group):
    comp, t, expected = _compressor(monkeypatch, group=group)
    assert expected() == [10] * 10                              # counts of the caller's own: as the descriptor says
    comp.run([(t, t, t)] * 6)                                   # one update, after four layers
    assert expected() == [10, 10, 10, 10, 64, 64, 10 + 54 * 2 // 6, 10, 64, 10 + 54 // 2]
    comp.select(1)
    assert expected()[:4] == [10, 64, 10, 10]
    comp.rebalance(4)
    assert expected()[:6] == [10, 10, 10, 10, 64, 64]


@pytest.mark.parametrize("schedule", ["fixed", "pyramid", "recent"])
def test_preset_budgets_cut_every_layer(monkeypatch, schedule):
    comp, t, expected = _compressor(monkeypatch, schedule=schedule)
    comp.run([(t, t, t)] * 6)
    assert expected() == [10] * 10
