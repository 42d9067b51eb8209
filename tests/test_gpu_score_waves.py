"""The second scoring sweep with keys owned by wavefronts (score_waves.h): ends of tiles, chunks and rounds of wavefronts, both row
widths, long chunks of many tiles, layers that follow each other in one call, token-major keys. Against float64."""
import math

import pytest
import torch

from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor

pytestmark = pytest.mark.gpu


def _cfg(Hq, Hkv, w, seqlens, L=1, P=7):
    return W.Workload("waves", L=L, Hq=Hq, Hkv=Hkv, d=128, seqlens=seqlens, dtype="bf16", w=w, P=P, mean_budget=8, layer_max=16,
                      interval=1, seed=0)


def _inputs(cfg, seed=3):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    make = lambda *s: torch.randn(s, generator=gen, device="cuda")
    return [(make(cfg.n_seqs, cfg.Hq, cfg.w, 128).to(torch.bfloat16), make(cfg.Hkv, cfg.total_tokens, 128).to(torch.bfloat16))
            for _ in range(cfg.L)]


def _check(cfg, got, q, k):
    """got [Hkv][T] against the scores in float64. A logit of y powers of two is rounded at 2^-24 y three times (product, its
    difference to the normaliser, the normaliser): that, four times over, and 16 for the sums, bounds the relative error."""
    rows = cfg.G * cfg.w
    for s in range(cfg.n_seqs):
        a, b = int(cfg.cu_seqlens[s]), int(cfg.cu_seqlens[s + 1])
        n = b - a - cfg.w
        assert torch.isneginf(got[:, max(a, b - cfg.w):b]).all() or n <= 0
        if n <= 0:
            continue
        for h in range(cfg.Hkv):
            x = q[s, h * cfg.G:(h + 1) * cfg.G].double().reshape(rows, 128) @ k[h, a:b].double().T / math.sqrt(128.0)
            seen = torch.arange(b - a, device="cuda")[None, :] <= n + (torch.arange(rows, device="cuda") % cfg.w)[:, None]
            y = float(x.abs().max()) / math.log(2.0)
            p = torch.softmax(x.masked_fill(~seen, -math.inf), dim=1).sum(0)[:n]
            half = cfg.P // 2
            ref = torch.nn.functional.max_pool1d(p[None, None], cfg.P, stride=1, padding=half)[0, 0]
            err = (got[h, a:a + n].double() - ref).abs() / ref.clamp_min(1e-30)
            assert float(err.max()) <= 4.0 * (3.0 * y + 16.0) * 2.0 ** -24, (s, h, float(err.max()), y)


@pytest.mark.parametrize("Hq,Hkv,w", [(2, 2, 8), (4, 2, 32), (6, 3, 31)])
@pytest.mark.parametrize("seqlens", [(39,), (65,), (255,), (263,), (518,), (1057,), (2079, 40, 7, 300)])
def test_edges_of_tiles_up_to_64_rows(Hq, Hkv, w, seqlens):
    cfg = _cfg(Hq, Hkv, w, seqlens)
    comp = Compressor(cfg, keep_cache=False)
    q, k = _inputs(cfg)[0]
    comp.score(0, q, k)
    _check(cfg, comp.scores[0], q, k)


# Long chunks: enough heads and tokens that a workgroup gets 1024 keys and more
@pytest.mark.parametrize("Hq,Hkv,w,seqlens", [(32, 8, 32, (32768,)), (24, 8, 32, (32741,)), (32, 8, 32, (65600,)),
                                              (64, 16, 32, (9000, 12001, 300)), (16, 8, 32, (40007,))])
def test_long_chunks(Hq, Hkv, w, seqlens):
    cfg = _cfg(Hq, Hkv, w, seqlens, L=3)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    layers = _inputs(cfg)
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
    many.score_layers(0, [x[0] for x in layers], [x[1] for x in layers])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    k_tm = layers[2][1].transpose(0, 1).contiguous()                     # token-major
    one.score(1, layers[2][0], k_tm, stride_token=cfg.Hkv * 128, stride_head=128)
    assert torch.equal(one.scores[1].view(torch.int32), many.scores[2].view(torch.int32))
    _check(cfg, many.scores[0], *layers[0])
    _check(cfg, many.scores[2], *layers[2])
