"""The rows behind the packed cache: zeros from the first block that does not fit (or the last row) to the capacity, every
other row as dkv_pack_cache wrote it; both head sizes and element types, capacities on both sides of the block borders."""
import pytest
import torch

from paper_2412_14838_amd import dkv
from paper_2412_14838_amd import workloads as W
from paper_2412_14838_amd.pipeline import Compressor

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "f32")])
def test_tail_of_the_packed_cache_is_zero(d, dtype):
    cfg = W.Workload("pack", L=5, Hq=3, Hkv=3, d=d, seqlens=(300, 16, 7, 900), dtype=dtype, w=16, P=7, mean_budget=20, layer_max=64,
                     interval=5, seed=1)
    comp = Compressor(cfg)
    comp.kb.normal_()
    comp.vb.normal_()
    gen = torch.Generator(device="cuda").manual_seed(3)
    comp.counts.copy_(torch.randint(0, 65, comp.counts.shape, generator=gen, device="cuda", dtype=torch.int32))
    strides = (cfg.n_seqs * cfg.Hkv * comp.slots * d, cfg.Hkv * comp.slots * d, comp.slots * d)

    def pack(capacity, tail):
        kp, vp = (torch.full((capacity, d), 7.0, dtype=comp.tdtype, device="cuda") for _ in range(2))
        off = torch.empty(cfg.n_seqs * cfg.L + 1, dtype=torch.int64, device="cuda")
        dkv.dkv_pack_cache(comp.desc, comp.cu, comp.counts, comp.kb, comp.vb, *strides, kp, vp, capacity, off)
        if tail:
            dkv.dkv_pack_zero_tail(comp.desc, off, kp, vp, capacity)
        torch.cuda.synchronize()
        return kp, vp, off.tolist()

    total = pack(1, False)[2][-1]
    off = pack(1, False)[2]
    for capacity in sorted({1, off[1] - 1, off[1], off[1] + 1, off[7], off[12] + 5, total - 1, total, total + 1, total + 70000}):
        end = max(o for o in off if o <= capacity)
        for raw, done in zip(pack(capacity, False)[:2], pack(capacity, True)[:2]):
            assert torch.equal(raw[:end], done[:end]) and (raw[end:] == 7).all() and (done[end:] == 0).all(), capacity


@pytest.mark.parametrize("n_seqs,L", [(1, 1), (64, 1), (13, 5), (1300, 4)])
def test_first_block_left_out_among_many(n_seqs, L):
    """The tail starts at the last offset within the capacity, whatever the number of blocks (one, 64, 65, thousands)."""
    cfg = W.Workload("many", L=L, Hq=1, Hkv=1, d=64, seqlens=(30,) * n_seqs, dtype="bf16", w=16, P=7, mean_budget=4, layer_max=8,
                     interval=1, seed=1)
    desc = dkv.desc_from_workload(cfg)
    gen = torch.Generator().manual_seed(n_seqs)
    off = torch.cat([torch.zeros(1, dtype=torch.int64), torch.randint(1, 4, (n_seqs * L,), generator=gen).cumsum(0)])
    dev = off.cuda()
    total, n = int(off[-1]), n_seqs * L
    for b in sorted({0, 1, n // 64, n // 2, n - 1, n} & set(range(n + 1))):
        for capacity in sorted({max(int(off[b]) + x, 1) for x in (-1, 0, 1)} | {total + 9}):
            k, v = (torch.full((capacity, cfg.d), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(2))
            dkv.dkv_pack_zero_tail(desc, dev, k, v, capacity)
            torch.cuda.synchronize()
            end = int(off[off <= capacity].max())
            for t in (k, v):
                assert (t[:end] == 7).all() and (t[end:] == 0).all(), (b, capacity)
