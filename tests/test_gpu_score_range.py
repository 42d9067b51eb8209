"""Scores of keys and queries at the upper end of their type's range: fills with the lowest value, -inf, large elements
whose products are ordinary, and ordinary elements whose logits are large. A logit of -inf (or far below the others) has no
weight; nothing else may notice. Of logits of 1e7 and more one key takes all of a row's weight.

Tolerance: as in test_gpu_score_tiles.py (the products of the large elements add at most a few units to the sum of the
absolute products there)."""
import numpy as np
import pytest
import torch

from oracle import dkv_oracle as O
from paper_2412_14838_amd import dkv as D
from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor, to_device

pytestmark = pytest.mark.gpu
RTOL = 1.3e-4
LARGEST = {"f32": float(np.finfo(np.float32).max), "bf16": float.fromhex("0x1.fep127")}


def _place(kind, cfg, data, largest):
    """Changes head 0 of every layer's data: positions inside a chunk, on both sides of a chunk border, next to the window
    and in it."""
    q, k = data["q_win"], data["k"]
    G, (j1, j2) = cfg.G, (5, cfg.d - 3)
    if kind.endswith("key"):
        q[:, :G] = np.abs(q[:, :G]) + np.float32(0.125)
    if kind in ("lowest_element", "minus_inf_element"):
        q[:, :G, :, j1] = np.abs(q[:, :G, :, j1]) + np.float32(0.125)
    if kind == "opposed":                                      # products past the range on both sides, the lower one larger
        q[:, :G, :, j1], q[:, :G, :, j2] = 2.0, -1.5
    if kind == "large_k":
        q[:, :G, :, j1] *= np.float32(2.0 / largest)
    if kind == "large_q":
        q[:, :G, :, j1] = largest
        k[0, :, j1] *= np.float32(2.0 / largest)
        return
    if kind.startswith("logits"):
        q[:, :G] *= np.float32(kind.split("_")[1])
        return
    for s in range(cfg.n_seqs):
        S, b = cfg.seqlens[s], int(cfg.cu_seqlens[s])
        for pos in (3, 250, 255, 256, 259, S - cfg.w - 1, S - 2):
            if 0 <= pos < S:
                row = k[0, b + pos]
                if kind == "lowest_element":
                    row[j1] = -largest
                elif kind == "lowest_key":
                    row[:] = -largest
                elif kind == "minus_inf_element":
                    row[j1] = -np.inf
                elif kind == "minus_inf_key":
                    row[:] = -np.inf
                elif kind == "opposed":
                    row[j1] = row[j2] = -largest
                elif kind == "large_k":
                    row[j1] = largest


KINDS = ["lowest_element", "lowest_key", "minus_inf_element", "minus_inf_key", "opposed", "large_k", "large_q", "logits_1e7",
         "logits_1e12"]
# (2 / largest, the factor of large_q, is a bf16 number of few bits: its products are not ordinary ones)
CASES = [(d, dtype, kind) for d, dtype in ((64, "f32"), (128, "f32"), (64, "bf16")) for kind in KINDS if (dtype, kind) != ("bf16", "large_q")]


@pytest.mark.parametrize("d,dtype,kind", CASES)
def test_scores_at_the_end_of_the_range(d, dtype, kind):
    cfg = W.Workload("range", L=2, Hq=6, Hkv=2, d=d, seqlens=(700, 262, 300), dtype=dtype, w=12, P=7, mean_budget=32, layer_max=64,
                     interval=1, seed=41)
    data = [W.make_layer(cfg, l, with_v=False) for l in range(cfg.L)]
    for x in data:
        _place(kind, cfg, x, LARGEST[dtype])
        if dtype == "bf16":                                    # what the device will hold
            x["q_win"] = W.round_to_bf16(x["q_win"])
    dev = [to_device(cfg, x) for x in data]
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    for l in range(cfg.L):
        one.score(l, dev[l]["q_win"], dev[l]["k"])
    many.score_layers(0, [x["q_win"] for x in dev], [x["k"] for x in dev])
    lse = torch.zeros((cfg.n_seqs, cfg.Hq, cfg.w), dtype=torch.float32, device="cuda")
    one.row_lse(lse)                                           # of the layer scored last
    single = torch.empty_like(one.scores[0])
    D.dkv_score_window_lse(one.desc, dev[-1]["q_win"], dev[-1]["k"], cfg.d, cfg.total_tokens * cfg.d, one.cu, lse, single,
                           cfg.total_tokens)
    torch.cuda.synchronize()
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    cu = cfg.cu_seqlens
    found = [(l, one.scores[l].cpu().numpy()) for l in range(cfg.L)]
    if not kind.startswith("logits"):                          # an exported normaliser of 1e7 is a multiple of 1 or more
        found.append((cfg.L - 1, single.cpu().numpy()))
    for l, got in found:
        for s in range(cfg.n_seqs):
            n = cfg.seqlens[s] - cfg.w
            ref = O.score_window(data[l]["q_win"][s], data[l]["k"][:, cu[s]:cu[s + 1]], cfg.P)
            off = np.abs(got[:, cu[s]:cu[s] + n] - ref)
            assert np.isfinite(off).all() and (off <= RTOL * ref).all(), (l, s, off.max())
            assert np.isneginf(got[:, cu[s] + n:cu[s + 1]]).all()


@pytest.mark.parametrize("d", [64, 128])
def test_infinite_logits_and_nan_stay_in_their_head(d):
    """As softmax has it: a logit of +inf or NaN leaves no number in its (sequence, KV head), and every number in the others."""
    cfg = W.Workload("nan", L=1, Hq=4, Hkv=2, d=d, seqlens=(600, 300), dtype="f32", w=16, P=1, mean_budget=32, layer_max=64,
                     interval=1, seed=42)
    clean = W.make_layer(cfg, 0, with_v=False)
    for bad in (np.inf, np.nan):
        data = {"q_win": np.abs(clean["q_win"]), "k": clean["k"].copy()}
        data["k"][1, 600 + 20, 7] = bad
        dev, comp = to_device(cfg, data), Compressor(cfg, keep_cache=False)
        comp.score(0, dev["q_win"], dev["k"])
        torch.cuda.synchronize()
        got = comp.scores[0].cpu().numpy()
        for h, s in ((0, 0), (1, 0), (0, 1)):
            b, n = int(cfg.cu_seqlens[s]), cfg.seqlens[s] - cfg.w
            ref = O.score_window(data["q_win"][s], data["k"][:, b:b + cfg.seqlens[s]], cfg.P)[h]
            assert (np.abs(got[h, b:b + n] - ref) <= RTOL * ref).all()
        assert np.isnan(got[1, 600:600 + 300 - cfg.w]).all()


# bf16 at head size 128: the kernels that stream their keys through LDS, at numbers of rows (3 or 6 query heads x window) that leave
# some of their 64, 128 or 256 rows over. P = 1: a pooling window of several keys would hide a key without a number.
ROWS_128 = {"36_rows": (2, 3, 12, (700, 262, 300)), "72_rows": (2, 3, 24, (700, 262, 300)), "72_rows_long_chunks": (32, 3, 24, (8200,)),
            "144_rows": (2, 6, 24, (700, 262, 300))}


def _cfg_128(rows, L, seed):
    Hkv, G, w, seqlens = ROWS_128[rows]
    return W.Workload("range128", L=L, Hq=G * Hkv, Hkv=Hkv, d=128, seqlens=seqlens, dtype="bf16", w=w, P=1, mean_budget=32, layer_max=64,
                      interval=1, seed=seed)


@pytest.mark.parametrize("rows", list(ROWS_128))
@pytest.mark.parametrize("kind", ["lowest_element", "lowest_run", "lowest_key", "minus_inf_element", "minus_inf_key", "large_k"])
def test_bf16_scores_at_the_end_of_the_range_at_head_size_128(kind, rows):
    cfg = _cfg_128(rows, 2, 43)
    data = [W.make_layer(cfg, l, with_v=False) for l in range(cfg.L)]
    for x in data:
        _place(kind, cfg, x, LARGEST["bf16"])
        if kind == "lowest_run":                               # logits of -1e36 to -1e38 in all keys of some chunks, finite ones
            x["q_win"][:, :cfg.G, :, 5] = 0.125 * (1 + np.arange(cfg.w) % 7)
            for b, e in zip(cfg.cu_seqlens, cfg.cu_seqlens[1:]):
                x["k"][0, b + 256:e - cfg.w, 5] = -LARGEST["bf16"]
        x["q_win"] = W.round_to_bf16(x["q_win"])               # what the device will hold
    dev = [to_device(cfg, x) for x in data]
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    for l in range(cfg.L):
        one.score(l, dev[l]["q_win"], dev[l]["k"])
    many.score_layers(0, [x["q_win"] for x in dev], [x["k"] for x in dev])
    torch.cuda.synchronize()
    cu = cfg.cu_seqlens
    for l in range(cfg.L):
        got = one.scores[l].cpu().numpy()
        for s in range(cfg.n_seqs):
            n = cfg.seqlens[s] - cfg.w
            ref = O.score_window(data[l]["q_win"][s], data[l]["k"][:, cu[s]:cu[s + 1]], cfg.P)
            off = np.abs(got[:, cu[s]:cu[s] + n] - ref)
            assert np.isfinite(off).all() and (off <= RTOL * ref).all(), (l, s, off.max())
            assert np.isneginf(got[:, cu[s] + n:cu[s + 1]]).all()
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))


@pytest.mark.parametrize("rows", list(ROWS_128))
def test_bf16_infinite_logits_and_nan_stay_in_their_head_at_head_size_128(rows):
    cfg = _cfg_128(rows, 1, 44)
    clean = W.make_layer(cfg, 0, with_v=False)
    s = cfg.n_seqs - 1                                         # the last sequence, head 1
    cu, at = cfg.cu_seqlens, int(cfg.cu_seqlens[s])
    for bad in (np.inf, np.nan):
        data = {"q_win": np.abs(clean["q_win"]), "k": clean["k"].copy()}
        data["k"][1, at + 20, 7] = bad
        dev, comp = to_device(cfg, data), Compressor(cfg, keep_cache=False)
        comp.score(0, dev["q_win"], dev["k"])
        torch.cuda.synchronize()
        got = comp.scores[0].cpu().numpy()
        for q in range(cfg.n_seqs):
            n = cfg.seqlens[q] - cfg.w
            with np.errstate(invalid="ignore"):
                ref = O.score_window(data["q_win"][q], data["k"][:, cu[q]:cu[q + 1]], cfg.P)
            for h in range(cfg.Hkv):
                if (q, h) != (s, 1):
                    assert (np.abs(got[h, cu[q]:cu[q] + n] - ref[h]) <= RTOL * ref[h]).all(), (q, h)
        assert np.isnan(got[1, at:at + cfg.seqlens[s] - cfg.w]).all()
