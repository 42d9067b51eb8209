"""The decode attention of a call whose workgroups fit the device at once (one kernel) against the two kernels of larger
calls (the same bits) and against float64."""
import numpy as np
import pytest
import torch

from paper_2412_14838_amd.pipeline import Compressor
from paper_2412_14838_amd.workloads import Workload

pytestmark = pytest.mark.gpu

# rows of a cache block around the ends of tiles (32 rows), slabs (128) and turns of a workgroup (512); w window rows come first
EDGES = [0, 1, 31, 32, 33, 63, 95, 96, 97, 127, 128, 129, 223, 224, 225, 256, 383, 384, 479, 480, 481, 511, 512, 513, 991,
         992, 993, 1024, 1504, 1505, 2016, 2048]


@pytest.mark.parametrize("Hkv,G,d,seqlens,w,layer_max", [
    (8, 4, 128, (4000,), 32, 2048), (8, 1, 128, (4000,), 32, 513), (4, 7, 128, (2500,), 32, 256), (8, 16, 128, (2500,), 16, 500),
    (8, 2, 64, (2500, 2500), 8, 1024), (5, 3, 128, (20, 3000, 32, 33), 32, 97), (16, 5, 64, (40, 7), 16, 30),
])
def test_one_kernel_gives_the_bits_of_two(dkv, Hkv, G, d, seqlens, w, layer_max):
    L = len(EDGES)
    cfg = Workload("decode", L=L, Hq=Hkv * G, Hkv=Hkv, d=d, seqlens=seqlens, dtype="bf16", w=w, P=7,
                   mean_budget=max(layer_max // 4, 1), layer_max=layer_max, interval=4, seed=3)
    comp = Compressor(cfg, group=1)
    gen = torch.Generator(device="cuda").manual_seed(G * 1000 + layer_max)
    comp.kb.copy_(torch.randn(comp.kb.shape, generator=gen, device="cuda"))
    comp.vb.copy_(torch.randn(comp.vb.shape, generator=gen, device="cuda"))
    counts = np.zeros((cfg.n_seqs, L), np.int32)
    for s, S in enumerate(seqlens):
        counts[s] = np.minimum(np.roll(EDGES, s), max(min(S - w, layer_max), 0))
    comp.counts.copy_(torch.from_numpy(counts).reshape(comp.counts.shape))
    # peaked logits: q of size 2
    q = (2.0 * torch.randn((L, cfg.n_seqs, cfg.Hq, d), generator=gen, device="cuda")).to(torch.bfloat16)
    one = torch.full((L, cfg.n_seqs, cfg.Hq, d), float("nan"), device="cuda")
    one_lse = torch.full((L, cfg.n_seqs, cfg.Hq), float("nan"), device="cuda")
    two, two_lse = torch.full_like(one, float("nan")), torch.full_like(one_lse, float("nan"))
    dkv.dkv_profile_begin(2 * L + 2)
    for l in range(L):
        comp.decode_attention(l, q[l], one[l], one_lse[l])
    assert [name for name, _ in dkv.dkv_profile_end(2 * L + 2)] == ["decode"] * L            # one launch each
    assert L * cfg.n_seqs * Hkv * (d // 32) > 256            # more than the device's compute units: the other route
    dkv.dkv_profile_begin(4)
    comp.decode_attention_layers(0, L, q, two, two_lse)
    assert [name for name, _ in dkv.dkv_profile_end(4)] == ["decode"] * 2
    torch.cuda.synchronize()
    assert torch.equal(one, two) and torch.equal(one_lse, two_lse)
    kb = comp.kb.reshape(L, cfg.n_seqs, Hkv, -1, d).double()
    vb = comp.vb.reshape(L, cfg.n_seqs, Hkv, -1, d).double()
    for l in range(0, L, 5):
        for s, S in enumerate(seqlens):
            wq = min(S, w)
            k, v = (x[l, s, :, w - wq:w + int(counts[s, l])] for x in (kb, vb))
            logits = torch.matmul(q[l, s].double().reshape(Hkv, G, d), k.transpose(1, 2).contiguous()) / d ** 0.5
            want = torch.matmul(torch.softmax(logits, -1), v).reshape(cfg.Hq, d)
            # fp32 sums of up to 2080 weights that add up to one, P in two bf16 terms (2^-17): as the other decode tests
            assert (one[l, s].double() - want).abs().max() <= 2e-5 * max(1.0, float(want.abs().max())), (l, s)
            assert (one_lse[l, s].double() - torch.logsumexp(logits, -1).reshape(-1)).abs().max() <= 2e-5 * 10, (l, s)
