"""GPU parity of the update's passes over the scores where their workgroups' shares end or overflow: one to nine heads
(four share a workgroup), rows of one position, of a chunk of 8192 and one more or less, rows that start off a 16-byte
boundary, more equal scores at the threshold than a workgroup of the last scan collects, zero scores at the threshold,
updates whose thresholds lie in different top digits. Hit counts and budgets bit-exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import dkv_oracle as O
from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor

pytestmark = pytest.mark.gpu


def _scores(kind, cfg, rng):
    shape = (cfg.L, cfg.Hkv, cfg.total_tokens)
    A = np.abs(rng.standard_normal(shape)).astype(np.float32) + np.float32(1e-3)
    if kind == "plateau":
        A[rng.random(shape) < 0.4] = 8.0
    elif kind == "zeros":
        A[rng.random(shape) < 0.995] = 0.0
    elif kind == "scaled":                                    # every layer an eighth of the one before: the thresholds fall
        A *= np.float32(0.125) ** np.arange(cfg.L, dtype=np.float32)[::-1, None, None]
    return A


@pytest.mark.parametrize("kind", ["smooth", "plateau", "zeros", "scaled"])
@pytest.mark.parametrize("Hkv,seqlens", [(1, (8192 + 8, 9)), (3, (8191 + 8, 8193 + 8, 41)), (4, (1201,)), (5, (16384 + 9, 77)),
                                         (9, (333, 8, 2050))])
def test_update_scans_match_the_oracle(Hkv, seqlens, kind):
    cfg = W.Workload("scans", L=6, Hq=Hkv, Hkv=Hkv, d=64, seqlens=seqlens, dtype="bf16", w=8, P=7, mean_budget=40, layer_max=160,
                     interval=2, seed=1)
    A = _scores(kind, cfg, np.random.default_rng(7 * Hkv + len(kind)))
    cu = cfg.cu_seqlens
    for batch in (False, True):
        comp = Compressor(cfg, keep_cache=False)
        comp.scores.copy_(torch.from_numpy(A))
        comp.select_layers(0, cfg.L)
        if batch:
            comp.rebalance_batch(2, 3)
        else:
            for l in (2, 4, 6):
                comp.rebalance(l)
        torch.cuda.synchronize()
        hits, budgets = comp.hits_all.cpu().numpy(), comp.budgets_all.cpu().numpy()
        for slot, l in enumerate((2, 4, 6)):
            for s in range(cfg.n_seqs):
                pre = seqlens[s] - cfg.w
                if pre <= 0:
                    continue
                cnt, _, Zp = O.update_buffer_length([A[i][:, cu[s]:cu[s] + pre] for i in range(l)], cfg.layer_max, cfg.mean_budget, cfg.L)
                assert np.array_equal(hits[slot, s, :l], cnt), (batch, l, s)
                assert np.array_equal(budgets[slot, s, :l], np.minimum(Zp, 2**31 - 1)), (batch, l, s)


def _check_updates(cfg, A, done):
    for batch in (False, True):
        comp = Compressor(cfg, keep_cache=False)
        comp.scores.copy_(torch.from_numpy(A))
        comp.select_layers(0, cfg.L)
        if batch:
            comp.rebalance_batch(done[0], len(done))
        else:
            for l in done:
                comp.rebalance(l)
        torch.cuda.synchronize()
        hits, budgets = comp.hits_all.cpu().numpy(), comp.budgets_all.cpu().numpy()
        cu = cfg.cu_seqlens
        for slot, l in enumerate(done):
            for s in range(cfg.n_seqs):
                pre = cfg.seqlens[s] - cfg.w
                if pre <= 0:
                    continue
                cnt, _, Zp = O.update_buffer_length([A[i][:, cu[s]:cu[s] + pre] for i in range(l)], cfg.layer_max, cfg.mean_budget, cfg.L)
                assert np.array_equal(hits[slot, s, :l], cnt), (batch, l, s)
                assert np.array_equal(budgets[slot, s, :l], np.minimum(Zp, 2**31 - 1)), (batch, l, s)


# workgroups of four heads of 8192 positions (the mean length is more) and of two heads of 4096
@pytest.mark.parametrize("kind", ["smooth", "plateau", "zeros", "scaled"])
@pytest.mark.parametrize("Hkv,seqlens", [(6, (8193 + 8,)), (1, (16385 + 8,)), (2, (9, 24600)), (3, (4095 + 8, 4096 + 8, 4097 + 8)),
                                         (1, (8192,)), (8, tuple(30 + 11 * i for i in range(40))),
                                         (2, tuple((5 * i) % 61 + (3000 if i % 50 == 0 else 1) for i in range(150)))])
def test_both_shapes_of_workgroups(Hkv, seqlens, kind):
    cfg = W.Workload("shapes", L=4, Hq=Hkv, Hkv=Hkv, d=64, seqlens=seqlens, dtype="bf16", w=8, P=7, mean_budget=40, layer_max=160,
                     interval=2, seed=1)
    _check_updates(cfg, _scores(kind, cfg, np.random.default_rng(11 * Hkv + len(kind))), (2, 4))


@pytest.mark.parametrize("Hkv,chunk,sharing", [(4, 8192, 7168), (4, 8192, 7169), (2, 4096, 1792), (2, 4096, 1793)])
def test_as_many_elements_at_the_threshold_as_the_last_scan_collects(Hkv, chunk, sharing):
    cfg = W.Workload("cap", L=2, Hq=Hkv, Hkv=Hkv, d=64, seqlens=(chunk + 8,), dtype="bf16", w=8, P=7, mean_budget=sharing // 8, layer_max=1800,
                     interval=1, seed=1)
    rng = np.random.default_rng(sharing)
    A = np.full((cfg.L, cfg.Hkv, cfg.total_tokens), -np.inf, np.float32)
    for l in range(cfg.L):
        row = rng.uniform(0.1, 0.5, Hkv * chunk).astype(np.float32)
        where = rng.permutation(Hkv * chunk)
        # one value of the upper 22 bits, all of the last digit; above them some that the scan before has counted
        row[where[:sharing]] = (np.uint32(0x3F800400) + rng.integers(0, 1024, sharing).astype(np.uint32)).view(np.float32)
        row[where[sharing:sharing + 50]] = 3.0
        A[l, :, :chunk] = row.reshape(Hkv, chunk)
    _check_updates(cfg, A, (1, 2))


def test_scores_on_the_borders_of_the_digits():
    cfg = W.Workload("borders", L=6, Hq=5, Hkv=5, d=64, seqlens=(9000, 77, 300), dtype="bf16", w=8, P=7, mean_budget=40, layer_max=160,
                     interval=2, seed=1)
    rng = np.random.default_rng(3)
    top, mid = np.uint32(0x3F800000 >> 21), np.uint32(700)
    at = (top << np.uint32(21)) | (mid << np.uint32(10))
    values = np.array([top << 21, (top << 21) - 1, ((top + 1) << 21) - 1, (top + 1) << 21, at, at - 1, at + 1023, at + 1024, 1, 0], np.uint32)
    for most_common in range(len(values)):                     # the thresholds move through the borders
        p = np.full(len(values), 0.004)
        p[most_common] = 1 - p.sum() + p[most_common]
        A = values[rng.choice(len(values), (cfg.L, cfg.Hkv, cfg.total_tokens), p=p)].view(np.float32)
        _check_updates(cfg, A, (2, 4, 6))
