"""The second scoring sweep with keys owned by wavefronts (score_waves.h): ends of tiles, chunks and rounds of wavefronts, both row
widths, long chunks of many tiles, layers that follow each other in one call, token-major keys. Against float64."""
import math

import pytest
import torch

from paper_2412_14838_amd import dkv as D
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


def _n_chunks(cfg, q, k):
    """Chunks that a call cuts the keys into, from the row statistics [chunk][Hkv][rows padded to 64 or 128][2] that it leaves at the
    workspace's start."""
    comp = Compressor(cfg, keep_cache=False)
    comp.ws.fill_(255)                                                   # NaN
    T, pad = cfg.total_tokens, 64 if cfg.G * cfg.w <= 64 else 128
    D.dkv_score_window_stats(comp.desc, q, k, cfg.d, T * cfg.d, comp.cu, comp.scores[0], T, comp.ws)
    n = T // 256 + cfg.n_seqs
    stats = comp.ws.view(torch.float32)[:n * cfg.Hkv * pad * 2].view(n, cfg.Hkv, pad, 2)
    return int((~torch.isnan(stats[:, 0, 0, 0])).sum())


# A last chunk of fewer tiles than wavefronts (1, 2, 2 and 7 of 8 have one), behind 31 whole ones: the others only keep the barriers
@pytest.mark.parametrize("Hq,Hkv,w", [(32, 8, 32), (24, 8, 32), (40, 8, 13), (16, 8, 32)])
@pytest.mark.parametrize("last,P", [(1, 7), (33, 1), (40, 63), (224, 7)])
def test_wavefronts_without_keys(Hq, Hkv, w, last, P):
    cfg = _cfg(Hq, Hkv, w, (31 * 1024 + w + last,), L=3, P=P)
    layers = _inputs(cfg)
    assert _n_chunks(cfg, *layers[0]) == 32                              # of 1024 keys: of all multiples of 128 only that one gives 32
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
    many.score_layers(0, [x[0] for x in layers], [x[1] for x in layers])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    for l in (0, 2):
        _check(cfg, many.scores[l], *layers[l])


# Heads one by one have chunks of 256 keys, together of 1024: 65 to 128 rows take score_emit_mfma there and this kernel here. With the
# normalisers handed over nothing else depends on the chunk.
@pytest.mark.parametrize("Hq,w,P", [(32, 32, 7), (24, 32, 1), (40, 13, 63)])
@pytest.mark.parametrize("S", [31 * 1024 + 73, 32768])
def test_the_same_bits_as_the_sweep_of_shared_tiles(Hq, w, P, S):
    cfg = _cfg(Hq, 8, w, (S,), P=P)
    (q, k), G = _inputs(cfg)[0], Hq // 8
    assert _n_chunks(cfg, q, k) == 32
    comp = Compressor(cfg, keep_cache=False)
    comp.score(0, q, k)
    lse = torch.empty((1, Hq, w), device="cuda")
    comp.row_lse(lse)
    comp.score_from_lse(0, q, k, lse)
    for h in range(8):
        alone = _cfg(G, 1, w, (S,), P=P)
        q_h, k_h, lse_h = (x.contiguous() for x in (q[:, h * G:(h + 1) * G], k[h:h + 1], lse[:, h * G:(h + 1) * G]))
        assert _n_chunks(alone, q_h, k_h) == -(-S // 256)
        part = Compressor(alone, keep_cache=False)
        part.score_from_lse(0, q_h, k_h, lse_h)
        assert torch.equal(part.scores[0, 0].view(torch.int32), comp.scores[0, h].view(torch.int32)), h


@pytest.mark.parametrize("Hq,Hkv,w,seqlens,chunks", [(32, 8, 32, (32768,), 32), (24, 8, 32, (32741,), 32), (32, 8, 32, (65600,), 31),
                                                     (64, 16, 32, (9000, 12001, 300), 15), (16, 8, 32, (40007,), 32)])
def test_chunks_of_long_prompts(Hq, Hkv, w, seqlens, chunks):
    """What test_long_chunks goes by: chunks of 1024 (twice), 2176, 1536 and 1280 keys. Rows from 65 on need 1024 to come here."""
    cfg = _cfg(Hq, Hkv, w, seqlens)
    assert _n_chunks(cfg, *_inputs(cfg)[0]) == chunks
