"""Scores of 129 to 256 rows per KV head: every number of row tiles, partly filled ones, ends of tiles, chunks and rounds of wavefronts,
wavefronts without keys, layers that follow each other in one workgroup, batches, very long chunks. Against float64, with the bound of
test_gpu_score_waves; test_score_route_cpu.py has the kernels and cuts."""
import pytest
import torch

from paper_2412_14838_amd.pipeline import Compressor
from test_gpu_score_waves import _cfg, _check, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,w", [(3, 1, 43), (10, 2, 32), (6, 1, 31), (14, 2, 32), (7, 1, 29), (9, 1, 25), (8, 1, 32), (8, 2, 64)])
@pytest.mark.parametrize("seqlens", [(257,), (97, 290), (300, 66, 700, 65), (2100,), (4705,)])
def test_rows_and_edges(Hq, Hkv, w, seqlens):
    cfg = _cfg(Hq, Hkv, w, seqlens, L=3)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    layers = _inputs(cfg)
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
    many.score_layers(0, [x[0] for x in layers], [x[1] for x in layers])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    for l in (0, 2):
        _check(cfg, many.scores[l], *layers[l])


@pytest.mark.parametrize("Hq,Hkv,w,seqlens,L", [(28, 4, 32, (32768,), 3), (40, 8, 32, (16001,), 5), (16, 2, 32, (70000,), 4), (24, 4, 32, (9000, 20001), 2)])
def test_long_chunks(Hq, Hkv, w, seqlens, L):
    cfg = _cfg(Hq, Hkv, w, seqlens, L=L)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    layers = _inputs(cfg)
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
    many.score_layers(0, [x[0] for x in layers], [x[1] for x in layers])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    _check(cfg, many.scores[L - 1], *layers[L - 1])
    k_tm = layers[1][1].transpose(0, 1).contiguous()                     # token-major
    one.score(0, layers[1][0], k_tm, stride_token=cfg.Hkv * 128, stride_head=128)
    assert torch.equal(one.scores[0].view(torch.int32), many.scores[1].view(torch.int32))


# Batches of short sequences, several layers to a workgroup: query heads, KV heads, window, lengths, layers
BY_SHARED_TILES = [(16, 2, 32, (187,) * 100, 16), (14, 2, 32, (133, 40, 170, 33) * 20, 16), (12, 2, 32, (180, 161, 190) * 22, 16),
                   (64, 8, 32, (180,) * 16, 16), (16, 2, 32, (500, 1200, 333, 1, 900) * 7, 7), (28, 4, 32, (500,) * 50, 4)]
BY_WAVES = [(16, 2, 32, (130,) * 100, 8), (14, 2, 32, (500,) * 64, 16), (12, 2, 32, (90,) * 64, 16), (10, 2, 32, (130, 77) * 32, 16)]


@pytest.mark.parametrize("Hq,Hkv,w,seqlens,L", BY_SHARED_TILES + BY_WAVES)
@pytest.mark.parametrize("P", [1, 7, 63])
def test_batches_of_several_layers(Hq, Hkv, w, seqlens, L, P):
    """Whichever kernel takes them: the bits of the layers one by one, and as exact."""
    cfg = _cfg(Hq, Hkv, w, seqlens, L=L, P=P)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    layers = _inputs(cfg)
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
    many.score_layers(0, [x[0] for x in layers], [x[1] for x in layers])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    _check(cfg, many.scores[L - 1], *layers[L - 1])


@pytest.mark.parametrize("Hq,w", [(5, 32), (6, 32), (7, 31), (8, 32)])
@pytest.mark.parametrize("chunks", [1, 2, 3, 15, 16, 17, 31, 32, 33, 181])
def test_merges_of_chunks(Hq, w, chunks):
    """One head's chunks of 256 keys: merged by 256 threads in a call of one layer, by 512 in one of several."""
    cfg = _cfg(Hq, 1, w, (256 * chunks - 100,), L=2)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    layers = _inputs(cfg)
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
    many.score_layers(0, [x[0] for x in layers], [x[1] for x in layers])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    _check(cfg, one.scores[0], *layers[0])


# Three layers and more to a workgroup, the last chunk of `last` keys: 1, 2 or 3 of its 4 wavefronts have any. In the first sweep's cut (5
# layers in two shares, 3 in one) and in one of its own (11 in four). Rows: whole row tiles and partly filled ones.
LAYERS_IN_A_SHARE = [(t * Hkv, Hkv, w, w + S + last, L) for t in (5, 6, 7, 8) for w, last in ((32, 1), (31, 33), (32, 96))
                     for Hkv, L, S in (((4, 3, 79360) if t == 8 else (8, 5, 2560)), (4, 11, 23040))]


@pytest.mark.parametrize("Hq,Hkv,w,S,L", LAYERS_IN_A_SHARE)
def test_layers_after_each_other(Hq, Hkv, w, S, L):
    cfg = _cfg(Hq, Hkv, w, (S,), L=L)
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    layers = _inputs(cfg)
    lses = []
    for l, (q, k) in enumerate(layers):
        one.score(l, q, k)
        lses.append(torch.empty((1, Hq, w), device="cuda"))
        one.row_lse(lses[l])
    qs, ks = [x[0] for x in layers], [x[1] for x in layers]
    many.score_layers(0, qs, ks)
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    for l in (0, 1, L - 1):
        _check(cfg, many.scores[l], *layers[l])
    many.score_layers_from_lse(0, qs, ks, lses)
    for l in range(L):
        one.score_from_lse(l, *layers[l], lses[l])
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))


@pytest.mark.parametrize("Hq", [40, 64])
def test_first_sweep_of_very_long_chunks(Hq):
    """3136 keys: more than score_emit_mfma would have the LDS for."""
    cfg = _cfg(Hq, 8, 32, (100001,))
    comp = Compressor(cfg, keep_cache=False)
    q, k = _inputs(cfg)[0]
    comp.score(0, q, k)
    _check(cfg, comp.scores[0], q, k)
