"""Scoring of several layers in one call where the workgroups deal the layers out among themselves (prompts whose chunks do
not fill the device): bit for bit what one call per layer writes, for numbers of layers that do and do not divide, one to
two workgroups for all layers up to one per layer, and the single sweep over the exported normalisers."""
import numpy as np
import pytest
import torch

from oracle import dkv_oracle as O
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


@pytest.mark.parametrize("dtype,d,Hq,Hkv,w,n_seqs", [("bf16", 128, 8, 2, 16, 8), ("bf16", 128, 8, 2, 16, 9), ("bf16", 128, 4, 1, 32, 64),
                                                     ("bf16", 128, 4, 1, 32, 65), ("bf16", 128, 6, 2, 64, 150), ("f32", 128, 3, 1, 43, 70)])
def test_batches_on_both_sides_of_the_search_by_lanes(dtype, d, Hq, Hkv, w, n_seqs):
    """A workgroup finds its chunk among up to eight sequences one by one, among more by the lanes of a wavefront, 64 at a time:
    sequences of one and several chunks, shorter than the window, next to each other in every order. Against the oracle."""
    rng = np.random.default_rng(n_seqs)
    seqlens = tuple(int(x) for x in rng.choice([1, w, w + 1, w + 40, 256, 257, 700], n_seqs))
    cfg = W.Workload("batch", L=2, Hq=Hq, Hkv=Hkv, d=d, seqlens=seqlens, dtype=dtype, w=w, P=7, mean_budget=8, layer_max=16, interval=1,
                     seed=n_seqs, plant_normalize=True)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    data = [W.make_layer(cfg, l, with_v=False) for l in range(cfg.L)]
    dev = [to_device(cfg, x) for x in data]
    for comp in (one, many):
        comp.scores.fill_(9.0)
    for l in range(cfg.L):
        one.score(l, dev[l]["q_win"], dev[l]["k"])
    many.score_layers(0, [x["q_win"] for x in dev], [x["k"] for x in dev])
    torch.cuda.synchronize()
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    got, cu = one.scores.cpu().numpy(), cfg.cu_seqlens
    for l in range(cfg.L):
        for s in range(n_seqs):
            n = seqlens[s] - w
            if n <= 0:
                assert (got[l][:, cu[s]:cu[s + 1]] == 9.0).all()
                continue
            ref = O.score_window(data[l]["q_win"][s], data[l]["k"][:, cu[s]:cu[s + 1]], cfg.P)
            assert (np.abs(got[l][:, cu[s]:cu[s] + n] - ref) <= 2e-3 * ref).all(), (l, s)
            assert np.isneginf(got[l][:, cu[s] + n:cu[s + 1]]).all()
