"""GPU parity of the scoring kernels that keep their keys in registers (bf16 at head size 64, fp32), at the sizes where
their cuts fall: chunks of 256, 512 and 1024 keys and one more or less, row tiles of 32, more sequences than a wavefront
has lanes, the pooling halo of one and of two tiles.

Tolerance: a logit is a sum of d products, accumulated in fp32 in some order, so it is off by at most
d * 2^-24 * sum |q_j k_j| * scale; with N(0, 1) inputs and d <= 128 the sum is about 0.64 d and scale = d^-1/2, which
makes 5.5e-5. An exponential is off by as much relatively, its normaliser by no more: 1.1e-4 in all, and 2^-24 for each
of up to 256 rows added (1.5e-5). That is what sums of one sign could reach. fp32 elements are split into three bf16 terms
and six of the nine products are taken: a term or a product lost is off by 4e-6 and more and would still pass, so fp32 is
held to what roundings of either sign give. A logit and its row's normaliser, of 2^2 to 2^3, are each off by one or two 2^-24
of that (2e-7 to 5e-7): at most 4.9e-7 in the 2-norm of a head and 1.2e-6 in one score were seen here, and three times that is
allowed."""
import numpy as np
import pytest
import torch

from oracle import dkv_oracle as O
from paper_2412_14838_amd import dkv as D
from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor, to_device

pytestmark = pytest.mark.gpu
RTOL = 1.3e-4
F32_NORM, F32_MAX = 1.5e-6, 3.6e-6


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
    "chunks_of_512_in_two_rounds": _cfg("o", L=2, Hkv=16, Hq=16, seqlens=(16384 + 5,)),
    "chunks_of_1024": _cfg("p", Hkv=16, Hq=16, seqlens=(16384 - 5,)),
    # the window across the middle of a chunk (two stages of 512 keys) and inside its second stage
    "chunks_of_1024_ragged": _cfg("q", Hkv=8, Hq=8, seqlens=(10 * 1024 + 700, 9 * 1024 + 530, 8 * 1024 + 20)),
    # more tasks than compute units already in one layer, not a multiple of 256
    "many_tasks_f32_d128": _cfg("r", Hkv=8, Hq=32, d=128, seqlens=(5000, 3700, 1311), dtype="f32"),
    "many_tasks_f32_d64": _cfg("s", Hkv=8, Hq=24, w=16, P=5, seqlens=(9000, 1111, 64, 300), dtype="f32"),
    "many_tasks_f32_halo_of_two_tiles": _cfg("t", L=2, Hkv=8, Hq=16, P=63, seqlens=(9001,), dtype="f32"),
}
# chunk length of the kernels that keep their keys in registers, where a case is there for it (None: the vector ALU)
CHUNKS = {"rows_128_f32_d128": 256, "rows_129_f32_d128_vector_alu": None, "chunks_of_512": 512, "chunks_of_512_in_two_rounds": 512,
          "chunks_of_1024": 1024, "chunks_of_1024_ragged": 1024, "many_tasks_f32_d128": 256, "many_tasks_f32_d64": 256,
          "many_tasks_f32_halo_of_two_tiles": 256, "one_key_past_the_window": 256}


def _chunk_length(cfg, q, k, q_dev, k_dev, stride=None, stride_head=None):
    """Of the kernels that a call runs on, from the row statistics it leaves at the workspace's start, (maximum, sum) per row
    [chunk][Hkv][rows padded to 64, 128 or 256]: how many chunks there are, and whether the maxima are those of the logits
    times log2 e (registers) or of the logits (vector ALU)."""
    comp = Compressor(cfg, keep_cache=False)
    comp.ws.fill_(255)                                           # NaN
    T = cfg.total_tokens
    D.dkv_score_window_stats(comp.desc, q_dev, k_dev, stride or cfg.d, stride_head or T * cfg.d, comp.cu, comp.scores[0], T, comp.ws)
    torch.cuda.synchronize()
    rows = cfg.G * cfg.w
    pad = 64 if rows <= 64 else (128 if rows <= 128 else 256)
    n = T // 256 + cfg.n_seqs
    stats = comp.ws.view(torch.float32)[:n * cfg.Hkv * pad * 2].view(n, cfg.Hkv, pad, 2).cpu().numpy()
    written = int((~np.isnan(stats[:, 0, 0, 0])).sum())
    chunk = next((c for c in (256, 512, 1024) if sum(-(-S // c) for S in cfg.seqlens) == written), 0)
    largest = (k[0, :min(chunk, cfg.seqlens[0] - cfg.w + 1)].astype(np.float64) @ q[0, 0, 0].astype(np.float64)).max() / np.sqrt(cfg.d)
    factor = stats[0, 0, 0, 0] / largest
    assert min(abs(factor - 1), abs(factor - np.log2(np.e))) < 1e-3, factor
    return None if abs(factor - 1) < 1e-3 else chunk


@pytest.mark.parametrize("case", list(CASES))
def test_scores_match_the_oracle_alone_and_together(case):
    cfg = CASES[case]
    data = [W.make_layer(cfg, l, with_v=False) for l in range(cfg.L)]
    dev = [to_device(cfg, x) for x in data]
    if case in CHUNKS:
        assert _chunk_length(cfg, data[0]["q_win"], data[0]["k"], dev[0]["q_win"], dev[0]["k"]) == CHUNKS[case]
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
            off = got[:, cu[s]:cu[s] + n] - ref
            rel = np.abs(off) / ref
            assert rel.max() <= RTOL, (l, s, rel.max())
            if cfg.dtype == "f32":
                norm = np.sqrt((off ** 2).sum(axis=1) / (ref ** 2).sum(axis=1)).max()
                assert norm <= F32_NORM and rel.max() <= F32_MAX, (l, s, norm, rel.max())
            assert np.isneginf(got[:, cu[s] + n:cu[s + 1]]).all()


@pytest.mark.parametrize("d", [64, 128])
def test_every_product_of_the_split_counts(d):
    """Rows whose logits come from one product of terms alone, exactly: x = 2^a (1 + 2^-9 + 2^-18) has the terms 2^a, 2^(a-9)
    and 2^(a-18); a second element takes away what the other terms give. All logits are 16 m / sqrt(d), m = 0, 1, 2 by the key;
    without the product the row's would be 0 (or far off)."""
    cfg = W.Workload("terms", L=1, Hq=2, Hkv=1, d=d, seqlens=(700,), dtype="f32", w=6, P=1, mean_budget=32, layer_max=64, interval=1,
                     seed=1)
    m = (np.arange(700) % 3).astype(np.float64)
    two, three = 1 + 2.0 ** -9, 1 + 2.0 ** -9 + 2.0 ** -18
    q, k = np.zeros((12, d)), np.zeros((700, d))
    cases = [                                                    # (q elements, k elements / m)
        ([1.0], [16.0]),                                         # hi hi
        ([2.0 ** 8, -2.0 ** 8], [2.0 ** 5 * two, 2.0 ** 5]),     # hi mid
        ([2.0 ** 8 * two, -2.0 ** 8], [2.0 ** 5, 2.0 ** 5]),     # mid hi
        ([2.0 ** 11, -2.0 ** 11], [2.0 ** 11 * three, 2.0 ** 11 * two]),   # hi lo
        ([2.0 ** 11 * three, -2.0 ** 11 * two], [2.0 ** 11, 2.0 ** 11]),   # lo hi
        ([2.0 ** 11 * two, -2.0 ** 11, -2.0 ** 11 * two, 2.0 ** 11], [2.0 ** 11 * two, 2.0 ** 11 * two, 2.0 ** 11, 2.0 ** 11])]   # mid mid
    for half in range(2):                                        # in the first and in the last elements of the head
        at = 0 if half == 0 else d - 32
        for i, (a, b) in enumerate(cases):
            q[half * 6 + i, at:at + len(a)] = a
            k[:, at:at + len(b)] = m[:, None] * np.array(b)
            at += 4
    data = {"q_win": q.reshape(1, 2, 6, d).astype(np.float32), "k": k[None].astype(np.float32)}
    assert np.array_equal(data["q_win"].reshape(12, d), q) and np.array_equal(data["k"][0], k)       # all exact in fp32
    logits = k @ q.T
    assert np.array_equal(logits, np.repeat(16 * m[:, None], 12, axis=1))
    dev, comp = to_device(cfg, data), Compressor(cfg, keep_cache=False)
    comp.score(0, dev["q_win"], dev["k"])
    torch.cuda.synchronize()
    ref = O.score_window(data["q_win"][0], data["k"], cfg.P)
    got = comp.scores[0].cpu().numpy()[:, :694]
    assert (np.abs(got - ref) <= 4e-6 * ref).all()               # exact logits: the exponentials and sums of 12 rows and 700 keys


@pytest.mark.parametrize("d,dtype,rows", [(64, "bf16", 32), (64, "f32", 32), (128, "f32", 32)])
def test_token_strides_on_both_sides_of_the_32_bit_offsets(d, dtype, rows):
    """Keys 4 MiB apart take the vector ALU (1024 of them would pass 2^32 bytes), 16 bytes less the registers."""
    cfg = _cfg("stride", L=1, Hq=2, Hkv=2, d=d, w=rows, seqlens=(270, 40), dtype=dtype)
    size = 2 if dtype == "bf16" else 4
    data = W.make_layer(cfg, 0, with_v=False)
    dev = to_device(cfg, data)
    for stride_b, chunk in (((1 << 22) - 16, 256), (1 << 22, None)):
        stride = stride_b // size
        wide = torch.empty((cfg.total_tokens, stride), dtype=dev["k"].dtype, device="cuda")
        for h in range(cfg.Hkv):
            wide[:, 4096 * h:4096 * h + d] = dev["k"][h]
        assert _chunk_length(cfg, data["q_win"], data["k"], dev["q_win"], wide, stride, 4096) == chunk
        comp = Compressor(cfg, keep_cache=False)
        comp.score(0, dev["q_win"], wide, stride_token=stride, stride_head=4096)
        torch.cuda.synchronize()
        del wide
        got, cu = comp.scores[0].cpu().numpy(), cfg.cu_seqlens
        for s in range(cfg.n_seqs):
            n = cfg.seqlens[s] - cfg.w
            ref = O.score_window(data["q_win"][s], data["k"][:, cu[s]:cu[s + 1]], cfg.P)
            assert (np.abs(got[:, cu[s]:cu[s] + n] - ref) <= RTOL * ref).all()
