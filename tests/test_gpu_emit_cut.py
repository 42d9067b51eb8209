"""The second scoring sweep of a call over several layers cuts keys and layers in its own way: the bits are those of the layers one by one,
whatever divides into what: a layer to every share, or several and fewer in the last ones, with both sweeps and with the normalisers
handed over; both sides of the L2 rule; batches, which keep the first sweep's cut. test_score_route_cpu.py has the cuts."""
import pytest
import torch

from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor

pytestmark = pytest.mark.gpu


# New cuts of several layers to a share, unevenly: 10 shares of 3 or 2 layers and 3072 keys (128, 160, 224 rows); 64 rows: 8 of 3 or 2, 4 of 8
# or 7, 4 of 3 or 2
UNEVEN = [(28, 32, 8, 32, (9001,)), (28, 40, 8, 32, (9001,)), (28, 56, 8, 32, (9001,)), (23, 4, 2, 32, (12000,)), (31, 6, 3, 32, (16000,)),
          (11, 8, 4, 32, (12000,))]


@pytest.mark.parametrize("L,Hq,Hkv,w,seqlens", UNEVEN + [
    (2, 8, 8, 32, (5000,)), (7, 32, 8, 32, (5003,)), (5, 16, 8, 32, (9001,)), (31, 14, 2, 32, (7001,)), (32, 16, 4, 32, (4100, 40, 3000)),
    (13, 24, 8, 32, (3000, 1200, 33, 700)), (32, 8, 2, 16, (3333,)), (3, 64, 8, 32, (12000,))])
def test_layers_together_give_the_bits_of_each_alone(L, Hq, Hkv, w, seqlens):
    cfg = W.Workload("cut", L=L, Hq=Hq, Hkv=Hkv, d=128, seqlens=seqlens, dtype="bf16", w=w, P=7, mean_budget=8, layer_max=16, interval=1,
                     seed=0)
    gen = torch.Generator(device="cuda").manual_seed(11)
    make = lambda *s: torch.randn(s, generator=gen, device="cuda").to(torch.bfloat16)
    layers = [(make(cfg.n_seqs, Hq, w, 128), make(Hkv, cfg.total_tokens, 128)) for _ in range(L)]
    one, many, handed = (Compressor(cfg, keep_cache=False) for _ in range(3))
    lses = []
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
        lse = torch.empty((cfg.n_seqs, Hq, w), device="cuda")
        one.row_lse(lse)
        lses.append(lse)
    qs, ks = [x[0] for x in layers], [x[1] for x in layers]
    many.score_layers(0, qs, ks)
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    handed.score_layers_from_lse(0, qs, ks, lses)
    for l in (0, L // 2, L - 1):
        alone = Compressor(cfg, keep_cache=False)
        alone.score_from_lse(l, *layers[l], lses[l])
        assert torch.equal(alone.scores[l].view(torch.int32), handed.scores[l].view(torch.int32)), l
