"""Scoring of several layers in one call where the workgroups deal the layers out among themselves (prompts whose chunks do
not fill the device): bit for bit what one call per layer writes, for numbers of layers that do and do not divide, one to
two workgroups for all layers up to one per layer, and the single sweep over the exported normalisers."""
import pytest
import torch

from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,Hq,Hkv,w,seqlens", [(7, 8, 2, 16, (1200,)), (32, 2, 1, 8, (300,)), (5, 32, 8, 32, (4096,)),
                                                (5, 32, 8, 32, (4097,)), (3, 16, 8, 16, (8192,)), (9, 28, 4, 32, (2000, 40, 700)),
                                                (13, 8, 2, 64, (513, 255))])
def test_layers_dealt_out_to_workgroups_equal_per_layer_calls(L, Hq, Hkv, w, seqlens):
    cfg = W.Workload("shares", L=L, Hq=Hq, Hkv=Hkv, d=128, seqlens=seqlens, dtype="bf16", w=w, P=7, mean_budget=32, layer_max=64,
                     interval=1, seed=17)
    one, many, lse_many = (Compressor(cfg, keep_cache=False) for _ in range(3))
    data = [to_device(cfg, W.make_layer(cfg, l, with_v=False)) for l in range(L)]
    lses = []
    for comp in (one, many, lse_many):
        comp.scores.fill_(9.0)
    for l in range(L):
        one.score(l, data[l]["q_win"], data[l]["k"])
        lses.append(torch.empty((cfg.n_seqs, Hq, w), dtype=torch.float32, device="cuda"))
        one.row_lse(lses[-1])
    qs, ks = [x["q_win"] for x in data], [x["k"] for x in data]
    many.score_layers(0, qs, ks)
    lse_many.score_layers_from_lse(0, qs, ks, lses)
    torch.cuda.synchronize()
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    for l in range(L):
        one.score_from_lse(l, data[l]["q_win"], data[l]["k"], lses[l])
    torch.cuda.synchronize()
    assert torch.equal(one.scores.view(torch.int32), lse_many.scores.view(torch.int32))
