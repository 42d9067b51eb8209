"""The kernel and the cut that the host picks for a scoring call (bf16, head size 128), 256 compute units."""
import random
import shutil

import pytest

from score_route import sweeps
from test_gpu_emit_cut import UNEVEN
from test_gpu_score_wide import BY_SHARED_TILES, BY_WAVES, LAYERS_IN_A_SHARE

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def _call(Hq, Hkv, w, seqlens, L, given=0):
    return L, Hq, Hkv, w, list(seqlens), given


def test_second_sweep_of_more_than_128_rows(tmp_path):
    """Several layers to a workgroup and a short chunk: the kernel of shared tiles where its finer steps are worth more. One layer: never."""
    calls = [_call(*s, given=g) for s in BY_SHARED_TILES + BY_WAVES for g in (0, 1)] + [_call(*s[:4], 1) for s in BY_SHARED_TILES]
    found = [x["emit"] for x in sweeps(tmp_path, calls)]
    n = 2 * len(BY_SHARED_TILES)
    assert {(x["kernel"], *x["template"]) for x in found[:n]} == {("score_emit_mfma", 4, 2, 32)}
    for (L, Hq, Hkv, w, _, _), x in zip(calls[n:], found[n:]):
        assert (x["kernel"], x["template"]) == ("score_emit_waves", [-(-Hq // Hkv * w // 32), 1 if L == 1 else 32])


def test_every_call_fits_and_covers_its_layers(tmp_path):
    rng = random.Random(5)
    calls = []
    for _ in range(400):
        G, Hkv, n = rng.randint(1, 8), rng.choice([1, 2, 4, 8]), rng.choice([1, 1, 1, 2, 8, 40, 300])
        calls.append(_call(G * Hkv, Hkv, 32, [rng.randint(1, int(10 ** rng.uniform(1.6, 5.3 if n == 1 else 4))) for _ in range(n)], rng.randint(1, 32),
                           rng.randint(0, 1)))
    for (L, Hq, Hkv, w, seqlens, _), x in zip(calls, sweeps(tmp_path, calls)):
        for s in x.values():
            shares, each, T = s["grid"][2], abs(s["layers_each"]), sum(seqlens)
            assert s["lds"] <= 152 * 1024 and 256 <= s["chunk"] <= 4096 and s["layers"] == L
            assert shares * each <= 32 or s["layers_each"] < 0 or s["kernel"] == "score_stats_mfma"
            assert (shares - 1) * each < L <= shares * each                              # no share is empty, none is missing
            assert s["grid"][:2] == [-(-T // s["chunk"]) if len(seqlens) == 1 else T // s["chunk"] + len(seqlens), Hkv]


def test_chunks_of_one_head(tmp_path):
    """What test_merges_of_chunks goes by."""
    calls = [_call(Hq, 1, w, (256 * n - 100,), 1) for Hq, w in ((5, 32), (7, 31)) for n in (1, 33, 181)]
    assert {x["stats"]["chunk"] for x in sweeps(tmp_path, calls)} == {256}


def test_cuts_of_several_layers_to_a_share(tmp_path):
    """What test_layers_together_give_the_bits_of_each_alone goes by: the second sweep's own cut, shares of several layers, not all as many."""
    calls = [(*s[:4], list(s[4]), 0) for s in UNEVEN] + [(*s[:4], list(s[4]), 1) for s in UNEVEN if s[1] // s[2] > 2]
    for (L, *_), x in zip(calls, sweeps(tmp_path, calls)):
        x = x["emit"]
        assert x["kernel"] == "score_emit_waves" and x["layers_each"] > 1 and L % x["grid"][2] != 0


def test_layers_in_a_share_and_wavefronts_without_keys(tmp_path):
    """What test_layers_after_each_other goes by."""
    calls = [_call(Hq, Hkv, w, [S], L) for Hq, Hkv, w, S, L in LAYERS_IN_A_SHARE]
    cuts = set()
    for (L, Hq, Hkv, w, (S,), _), x in zip(calls, sweeps(tmp_path, calls)):
        x, tiles = x["emit"], -(-Hq // Hkv * w // 32)
        assert x["kernel"] == "score_emit_waves" and x["template"] == [tiles, 32] and abs(x["layers_each"]) >= 3
        last = (S - w) % x["chunk"]
        assert 1 <= last <= 96
        cuts.add((tiles, x["layers_each"] > 0, -(-last // 32)))
    assert cuts == {(t, own, n) for t in (5, 6, 7, 8) for own in (False, True) for n in (1, 2, 3)}


def test_first_sweep_of_very_long_chunks(tmp_path):
    calls = [_call(Hq, 8, 32, [100001], 1) for Hq in (40, 64)]
    assert [x[k]["chunk"] for x in sweeps(tmp_path, calls) for k in ("stats", "emit")] == [3136] * 4
