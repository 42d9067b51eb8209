"""GPU parity of the selection's upper-tail path (one histogram between a lower bound of the threshold and the row's
largest score) at the sizes and values where it can go wrong: rows of one position up to what a workgroup holds, k of
one and of two elements per thread and one more, ranges of a few ulps and of all exponents, infinities, zeros among the
winners, as many equal scores as the path takes and one more. Bit-exact against the oracle's stable sort."""
import numpy as np
import pytest
import torch

from oracle import dkv_oracle as O
from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor

pytestmark = pytest.mark.gpu


def _rows(n, k, rng):
    smooth = np.abs(rng.standard_normal(n)).astype(np.float32)
    pooled = np.maximum.reduce([np.roll(smooth, r) for r in range(-3, 4)])
    ulps = (np.uint32(0x3C000000) + rng.integers(0, 5000, n).astype(np.uint32)).view(np.float32)
    exponents = rng.integers(1, 0x7F800000, n).astype(np.uint32).view(np.float32)
    outliers = smooth * np.float32(1e-3)
    outliers[rng.integers(0, n, 3)] = [np.float32(1e30), np.float32("inf"), np.float32("inf")]
    sparse = np.zeros(n, np.float32)                          # zeros among the winners, unless k is small
    where = rng.permutation(n)[: max(k // 2, 1)]
    sparse[where] = smooth[where]
    out = [smooth, pooled, ulps, exponents, outliers, sparse]
    for equal in (4096 - k // 2, 4097 - k // 2):              # k / 2 larger scores, then a plateau that holds the threshold
        row = rng.uniform(0.001, 0.01, n).astype(np.float32)
        where = rng.permutation(n)
        row[where[: k // 2]] = rng.uniform(2.0, 3.0, min(k // 2, n)).astype(np.float32)
        row[where[k // 2:k // 2 + equal]] = 1.0
        out.append(row)
    return out


@pytest.mark.parametrize("layer_max", [1, 1024, 1025, 2048])
@pytest.mark.parametrize("longest", [1, 33, 1025, 2049, 8191, 8192, 8193, 16384, 16385, 32767, 32768])
def test_upper_tail_selection_is_the_stable_sort(longest, layer_max):
    rng = np.random.default_rng(100 * longest + layer_max)
    w = 16
    rows = _rows(longest, min(layer_max, longest), rng)
    cfg = W.Workload("tail", L=len(rows) // 2, Hq=2, Hkv=2, d=64, seqlens=(longest + w, max(longest // 3, 1) + w), dtype="bf16", w=w,
                     P=7, mean_budget=32, layer_max=layer_max, interval=1, seed=1)
    comp = Compressor(cfg, keep_cache=False)
    cu = cfg.cu_seqlens
    A = np.full((cfg.L, cfg.Hkv, cfg.total_tokens), -np.inf, np.float32)
    for i, row in enumerate(rows):
        for s in range(2):
            pre = cfg.seqlens[s] - w
            A[i // 2, i % 2, cu[s]:cu[s] + pre] = row[:pre]
    comp.scores.copy_(torch.from_numpy(A))
    comp.idx.fill_(-7)
    comp.select_layers(0, cfg.L)
    torch.cuda.synchronize()
    idx = comp.idx.cpu().numpy()
    for l in range(cfg.L):
        for s in range(2):
            ref = O.select_topk(A[l][:, cu[s]:cu[s] + cfg.seqlens[s] - w], layer_max)
            k = ref.shape[1]
            assert np.array_equal(idx[l, s][:, :k], ref), (l, s)
            assert (idx[l, s][:, k:] == -1).all()


@pytest.mark.parametrize("layer_max", [1, 1024, 1025, 2048])
@pytest.mark.parametrize("longest", [1, 1023, 1024, 1025, 2047, 2048, 2049, 5000, 20000, 32768])
def test_rows_whose_threads_share_the_largest_score(longest, layer_max):
    """Equal rows, rows of zeros, and rows in which each of the 1024 threads (position mod 1024) holds the largest score once
    or twice."""
    rng = np.random.default_rng(longest + layer_max)
    some = rng.uniform(0.1, 0.9, longest).astype(np.float32)
    once, twice = some.copy(), some.copy()
    once[:1024] = 1.0
    twice[:2048] = 1.0
    rows = [np.full(longest, 0.25, np.float32), np.zeros(longest, np.float32), once, twice]
    w = 16
    cfg = W.Workload("flat", L=len(rows), Hq=1, Hkv=1, d=64, seqlens=(longest + w,), dtype="bf16", w=w, P=7, mean_budget=1,
                     layer_max=layer_max, interval=1, seed=1)
    comp = Compressor(cfg, keep_cache=False)
    A = np.full((cfg.L, 1, cfg.total_tokens), -np.inf, np.float32)
    A[:, 0, :longest] = rows
    comp.scores.copy_(torch.from_numpy(A))
    comp.idx.fill_(-7)
    comp.select_layers(0, cfg.L)
    torch.cuda.synchronize()
    idx = comp.idx.cpu().numpy()
    for l in range(cfg.L):
        ref = O.select_topk(A[l][:, :longest], layer_max)
        assert np.array_equal(idx[l, 0][:, :ref.shape[1]], ref), l
        assert (idx[l, 0][:, ref.shape[1]:] == -1).all()


@pytest.mark.parametrize("layer_max", [100, 500, 1100])
def test_as_many_scores_at_the_threshold_as_are_compared_with_each_other(layer_max):
    """The number of elements at the threshold from which on the third digit is taken, and one more; equal scores, and scores
    that differ in their last bits."""
    cap = min(max(layer_max, 384), 768)
    rng = np.random.default_rng(layer_max)
    n, w = 9000, 16
    rows = []
    for equal in (cap, cap + 1):
        for spread in (1, 8):
            row = rng.uniform(0.001, 0.01, n).astype(np.float32)
            where = rng.permutation(n)
            row[where[:layer_max // 2]] = rng.uniform(2.0, 3.0, layer_max // 2).astype(np.float32)
            row[where[layer_max // 2:layer_max // 2 + equal]] = (np.uint32(0x3F800000) + rng.integers(0, spread, equal).astype(np.uint32)).view(np.float32)
            rows.append(row)
    cfg = W.Workload("share", L=len(rows), Hq=1, Hkv=1, d=64, seqlens=(n + w,), dtype="bf16", w=w, P=7, mean_budget=1,
                     layer_max=layer_max, interval=1, seed=1)
    comp = Compressor(cfg, keep_cache=False)
    A = np.full((cfg.L, 1, cfg.total_tokens), -np.inf, np.float32)
    A[:, 0, :n] = rows
    comp.scores.copy_(torch.from_numpy(A))
    comp.select_layers(0, cfg.L)
    torch.cuda.synchronize()
    idx = comp.idx.cpu().numpy()
    for l in range(cfg.L):
        assert np.array_equal(idx[l, 0], O.select_topk(A[l][:, :n], layer_max)), l
