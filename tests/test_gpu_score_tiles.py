"""GPU parity of the scoring kernels that keep their keys in registers (bf16 at head size 64, fp32), at the sizes where
their cuts fall: chunks of 256, 512 and 1024 keys and one more or less, row tiles of 32, more sequences than a wavefront
has lanes, the pooling halo of one and of two tiles.

Tolerance: a logit is a sum of d products, accumulated in fp32 in some order, so it is off by at most
d * 2^-24 * sum |q_j k_j| * scale; with N(0, 1) inputs and d <= 128 the sum is about 0.64 d and scale = d^-1/2, which
makes 5.5e-5. An exponential is off by as much relatively, its normaliser by no more: 1.1e-4 in all, and 2^-24 for each
of up to 256 rows added (1.5e-5)."""
import numpy as np
import pytest
import torch

from oracle import dkv_oracle as O
from paper_2412_14838_amd import dkv as D
from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor, to_device

pytestmark = pytest.mark.gpu
RTOL = 1.3e-4


def _cfg(name, **kw):
    base = dict(name=name, L=3, Hq=4, Hkv=2, d=64, seqlens=(1500,), dtype="bf16", w=32, P=7, mean_budget=32, layer_max=64,
                interval=1, seed=611, plant="loguniform", plant_lo=4, plant_hi=40, plant_normalize=True)
    base.update(kw)
    return W.Workload(**base)


CASES = {
    "one_key_past_the_window": _cfg("a", seqlens=(33, 32, 34)),
    "chunk_edges": _cfg("b", seqlens=(255, 256, 257, 511, 512, 513, 1023, 1024, 1025)),
    "chunk_edges_f32": _cfg("c", seqlens=(255, 256, 257, 511, 512, 513), dtype="f32"),
    "window_across_a_chunk": _cfg("d", seqlens=(256 + 10, 1024 + 31, 2048 + 1), w=48, Hq=2),
    "rows_1": _cfg("e", w=1, Hq=2, seqlens=(300, 2)),
    "rows_33": _cfg("f", w=11, Hq=6, seqlens=(700,)),
    "rows_224_f32": _cfg("g", w=32, Hq=14, seqlens=(600,), dtype="f32"),
    "rows_256": _cfg("h", w=64, Hq=8, seqlens=(600, 900)),
    "rows_128_f32_d128": _cfg("i", w=32, Hq=8, d=128, seqlens=(600, 257), dtype="f32"),
    "rows_129_f32_d128_vector_alu": _cfg("j", w=43, Hq=6, d=128, seqlens=(400,), dtype="f32"),
    "halo_of_two_tiles": _cfg("k", P=63, seqlens=(1100, 300)),
    "halo_of_two_tiles_f32": _cfg("l", P=35, Hq=16, w=32, seqlens=(1100,), dtype="f32"),
    "more_sequences_than_lanes": _cfg("m", L=2, seqlens=tuple(40 + (37 * i) % 300 for i in range(131))),
    "chunks_of_512": _cfg("n", L=2, Hkv=8, Hq=8, seqlens=(12000,)),
    "chunks_of_1024": _cfg("o", L=2, Hkv=16, Hq=16, seqlens=(16384 + 5,)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_scores_match_the_oracle_alone_and_together(case):
    cfg = CASES[case]
    data = [W.make_layer(cfg, l, with_v=False) for l in range(cfg.L)]
    dev = [to_device(cfg, x) for x in data]
    one, many = Compressor(cfg, keep_cache=False), Compressor(cfg, keep_cache=False)
    for c in (one, many):
        c.scores.fill_(7.0)
    for l in range(cfg.L):
        one.score(l, dev[l]["q_win"], dev[l]["k"])
    many.score_layers(0, [x["q_win"] for x in dev], [x["k"] for x in dev])
    lse = torch.zeros((cfg.n_seqs, cfg.Hq, cfg.w), dtype=torch.float32, device="cuda")
    one.row_lse(lse)                                             # of the layer scored last
    single = torch.full_like(one.scores[0], 7.0)
    D.dkv_score_window_lse(one.desc, dev[-1]["q_win"], dev[-1]["k"], cfg.d, cfg.total_tokens * cfg.d, one.cu, lse, single,
                           cfg.total_tokens)
    torch.cuda.synchronize()
    assert torch.equal(one.scores.view(torch.int32), many.scores.view(torch.int32))
    cu = cfg.cu_seqlens
    for l, got in [(l, one.scores[l].cpu().numpy()) for l in range(cfg.L)] + [(cfg.L - 1, single.cpu().numpy())]:
        for s in range(cfg.n_seqs):
            n = cfg.seqlens[s] - cfg.w
            if n <= 0:
                assert (got[:, cu[s]:cu[s + 1]] == 7.0).all()    # a sequence without a prefix is left alone
                continue
            ref = O.score_window(data[l]["q_win"][s], data[l]["k"][:, cu[s]:cu[s + 1]], cfg.P)
            rel = np.abs(got[:, cu[s]:cu[s] + n] - ref) / ref
            assert rel.max() <= RTOL, (l, s, rel.max())
            assert np.isneginf(got[:, cu[s] + n:cu[s + 1]]).all()
