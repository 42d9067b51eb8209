"""Timed cases of the prefill compression and of the decoding over its cache, through the package's public calls.

A case is a plain dict: the shape of a model's attention (layers L, query heads Hq, KV heads Hkv, head size d, element
type), the lengths of the sequences in the batch, the method's parameters (window w, pooling P, mean and maximal budget,
update interval) and what is run:

    prefill   Algorithm 1 over all layers, then the first new token's attention over the compressed cache.
              group 1: layer by layer, as a model that frees a layer's keys at once calls it; group 0: as many layers
              per call as the library takes. lse: the caller hands over the row normalisers its attention kernel holds.
    compact   selection, budget updates, compaction and the tight packing, for a caller that already holds the scores.
    decode    one new token per sequence, layer after layer, as an ordinary decoder does it.

The inputs follow workloads.py: Q, K, V ~ N(0, 1), some keys per layer ("heavy" positions, in short runs) pulled toward
the mean window query of their head, so that scores have the peaks of a long prompt and the layers' budgets differ.
"""
from __future__ import annotations

import math

import torch

from paper_2412_14838_amd import dkv
from paper_2412_14838_amd.pipeline import Compressor, default_group
from paper_2412_14838_amd.workloads import Workload, standard_configs


def _case(name, cfg, what="prefill", group=0, lse=False, schedule="dynamic"):
    return {"name": name, "what": what, "L": cfg.L, "Hq": cfg.Hq, "Hkv": cfg.Hkv, "d": cfg.d, "dtype": cfg.dtype,
            "seqlens": ",".join(str(s) for s in cfg.seqlens), "w": cfg.w, "P": cfg.P, "mean_budget": cfg.mean_budget,
            "layer_max": cfg.layer_max, "interval": cfg.interval, "group": group, "lse": lse, "schedule": schedule}


def listed():
    std = standard_configs()
    tiny, m8k, m32k = std["tiny"], std["llama3_8b_8k"], std["mistral_7b_32k"]
    extreme, ragged = std["qwen2_7b_32k_extreme"], std["ragged_batch8"]
    return [
        # the smallest call: four layers of a 1K prompt in fp32, bound by launches and latency
        _case("tiny_f32_1k", tiny),
        # one new token over the 32 compressed layers of a 32K prompt: what a user waits for per token
        _case("decode_32k", m32k, "decode"),
        # Algorithm 1's own order inside a model's forward pass, at the two context lengths of the paper's table
        _case("layerwise_8k", m8k, group=1),
        _case("layerwise_32k", m32k, group=1),
        # fp32 weights (accuracy checks, small deployments)
        _case("prefill_f32_8k", m8k.with_(L=8, seqlens=(8192,), dtype="f32")),
        # the other head size the library takes, as small models have it
        _case("prefill_d64_16k", m8k.with_(L=16, Hq=16, Hkv=8, d=64, seqlens=(16384,), mean_budget=256, layer_max=1024)),
        # selection, updates and compaction alone: a caller that scores inside its own attention kernel, ragged batch
        _case("compact_ragged", ragged, "compact"),
        # the main case: all layers of a 32K prompt, as many as a call takes
        _case("prefill_32k", m32k),
        # the same with the normalisers handed over (one sweep over the keys)
        _case("prefill_32k_lse", m32k, lse=True),
        # seven query heads per KV head, four KV heads, a very small budget
        _case("prefill_32k_group7", extreme),
        # a serving batch of eight prompts of different lengths
        _case("prefill_ragged8", ragged),
        # long context: rows too long for one workgroup's selection
        _case("prefill_128k", m32k.with_(L=8, seqlens=(131072,))),
    ]


_MOST_KEYS = 32 * 8 * 32768 * 128          # key elements of the largest listed case
_MOST_F32 = 8 * 8 * 8192 * 128             # of the largest fp32 one
_MOST_D64 = 16 * 8 * 16384 * 64            # of the largest one at head size 64


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["prefill"] * 7 + ["compact", "decode"])
    kind = rng.choice(["bf16"] * 6 + ["bf16_d64", "f32"])
    d = 64 if kind == "bf16_d64" or (kind == "f32" and rng.random() < 0.5) else 128
    dtype = "f32" if kind == "f32" else "bf16"
    Hkv = rng.choice([2, 4, 8, 8])
    w = rng.choice([8, 16, 32, 32, 32, 64])
    G = rng.choice([g for g in (1, 2, 4, 4, 5, 7, 8) if g * w <= 256])
    most = _MOST_F32 if kind == "f32" else (_MOST_D64 if d == 64 else _MOST_KEYS)
    n_seqs = rng.choice([1, 1, 1, 2, 4, 8])
    longest = 131072 if d == 128 and dtype == "bf16" else 16384
    tokens = _log(rng, 1024 * n_seqs, min(longest, most // (Hkv * d)))
    shares = [rng.uniform(0.4, 1.6) for _ in range(n_seqs)]
    lens = [max(w + 200, int(tokens * s / sum(shares))) for s in shares]
    L = rng.choice([4, 8, 16, 28, 32])
    while L > 4 and L * Hkv * d * sum(lens) > most:
        L //= 2
    layer_max = _log(rng, 96, 2048)
    schedule = rng.choice(["dynamic"] * 4 + ["pyramid"]) if what == "prefill" else "dynamic"
    group = 1 if schedule != "dynamic" or rng.random() < 0.3 else 0
    return {"what": what, "L": L, "Hq": Hkv * G, "Hkv": Hkv, "d": d, "dtype": dtype,
            "seqlens": ",".join(str(s) for s in lens), "w": w, "P": rng.choice([1, 3, 5, 7, 7, 7, 9, 13]),
            "mean_budget": max(32, layer_max // rng.choice([2, 4, 4])), "layer_max": layer_max,
            "interval": rng.choice([2, 4, 4]), "group": group, "lse": what == "prefill" and group == 0 and rng.random() < 0.2,
            "schedule": schedule}


def _cfg(case) -> Workload:
    return Workload("case", L=case["L"], Hq=case["Hq"], Hkv=case["Hkv"], d=case["d"],
                    seqlens=tuple(int(s) for s in case["seqlens"].split(",")), dtype=case["dtype"], w=case["w"],
                    P=case["P"], mean_budget=case["mean_budget"], layer_max=case["layer_max"],
                    interval=case["interval"], seed=0)


def _layers(cfg, gen, tdtype, with_v=True):
    """(q_win, k, v) of every layer, on the GPU."""
    T, cu = cfg.total_tokens, cfg.cu_seqlens
    out = []
    for _ in range(cfg.L):
        q = torch.randn((cfg.n_seqs, cfg.Hq, cfg.w, cfg.d), generator=gen, device="cuda").to(tdtype)
        k = torch.randn((cfg.Hkv, T, cfg.d), generator=gen, device="cuda")
        heavy = int(math.exp(float(torch.rand((), generator=gen, device="cuda")) * math.log(32.0)))      # runs of 8 keys
        for s in range(cfg.n_seqs):
            S = cfg.seqlens[s]
            mean_q = q[s].float().reshape(cfg.Hkv, cfg.G * cfg.w, cfg.d).mean(dim=1)
            toward = mean_q * (2.0 * math.sqrt(cfg.d) / mean_q.norm(dim=1, keepdim=True).clamp_min(1e-20))
            runs = torch.randint(0, max((S - cfg.w) // 8, 1), (heavy,), generator=gen, device="cuda")
            pos = (runs[:, None] * 8 + torch.arange(8, device="cuda")).reshape(-1).clamp_max(S - cfg.w - 1).unique()
            k[:, int(cu[s]) + pos] += toward[:, None, :]
        v = torch.randn((cfg.Hkv, T, cfg.d), generator=gen, device="cuda").to(tdtype) if with_v else None
        out.append((q, k.to(tdtype), v))
    return out


def prepare(case, seed):
    cfg = _cfg(case)
    tdtype = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    group = case["group"] or default_group(cfg)
    comp = Compressor(cfg, group=group, schedule=case["schedule"])
    layers = _layers(cfg, gen, tdtype)
    state = {"what": case["what"], "cfg": cfg, "comp": comp,
             "q_new": torch.randn((cfg.L, cfg.n_seqs, cfg.Hq, cfg.d), generator=gen, device="cuda").to(tdtype),
             "out": torch.zeros((cfg.L, cfg.n_seqs, cfg.Hq, cfg.d), dtype=torch.float32, device="cuda"),
             "lse_out": torch.zeros((cfg.L, cfg.n_seqs, cfg.Hq), dtype=torch.float32, device="cuda")}
    if case["what"] == "decode":
        comp.run(layers)                      # the decoder holds the compressed cache, not the prompt's keys
        return state
    state["layers"] = layers
    if case["what"] == "compact":
        for l0 in range(0, cfg.L, group):
            part = layers[l0:l0 + group]
            comp.score_layers(l0, [x[0] for x in part], [x[1] for x in part])
        state["packed_rows"] = cfg.n_seqs * cfg.L * cfg.Hkv * (cfg.w + cfg.mean_budget)
    if case["lse"]:
        scratch = torch.empty_like(comp.scores[0])
        state["lses"] = torch.empty((cfg.L, cfg.n_seqs, cfg.Hq, cfg.w), dtype=torch.float32, device="cuda")
        for l, (q, k, _) in enumerate(layers):
            dkv.dkv_score_window_stats(comp.desc, q, k, cfg.d, cfg.total_tokens * cfg.d, comp.cu, scratch,
                                       cfg.total_tokens, comp.ws)
            comp.row_lse(state["lses"][l])
    return state


def _after_scores(comp, cfg, layers, l0, n):
    """Selection, updates and compaction of layers l0 .. l0 + n - 1, whose scores are there."""
    comp.select_layers(l0, n)
    done = [l + 1 for l in range(l0, l0 + n) if (l + 1) % cfg.interval == 0]
    for i in range(0, len(done), dkv.DKV_MAX_UPDATES):
        part = done[i:i + dkv.DKV_MAX_UPDATES]
        comp.rebalance_batch(part[0], len(part))
    comp.gather_layers(l0, [x[1] for x in layers[l0:l0 + n]], [x[2] for x in layers[l0:l0 + n]])


def run(state):
    comp, cfg = state["comp"], state["cfg"]
    if state["what"] == "decode":
        for l in range(cfg.L):
            comp.decode_attention(l, state["q_new"][l], state["out"][l], state["lse_out"][l])
        return {"out": state["out"], "lse": state["lse_out"]}
    layers = state["layers"]
    if state["what"] == "compact":
        comp.epoch = 0                        # a pass of its own: no update history from the pass before
        for l0 in range(0, cfg.L, comp.group):
            _after_scores(comp, cfg, layers, l0, min(comp.group, cfg.L - l0))
        k_packed, v_packed, offsets = comp.pack(state["packed_rows"])
        return {"idx": comp.idx, "counts": comp.counts, "budgets": comp.budgets_all, "hits": comp.hits_all,
                "k": k_packed, "v": v_packed, "offsets": offsets}
    if "lses" in state:
        comp.epoch = 0
        for l0 in range(0, cfg.L, comp.group):
            part = layers[l0:l0 + comp.group]
            comp.score_layers_from_lse(l0, [x[0] for x in part], [x[1] for x in part],
                                       [state["lses"][l0 + i] for i in range(len(part))])
            _after_scores(comp, cfg, layers, l0, len(part))
    else:
        comp.run(layers)
    for l0 in range(0, cfg.L, dkv.DKV_MAX_SELECT_LAYERS):
        n = min(dkv.DKV_MAX_SELECT_LAYERS, cfg.L - l0)
        comp.decode_attention_layers(l0, n, state["q_new"][l0:l0 + n], state["out"][l0:l0 + n], state["lse_out"][l0:l0 + n])
    # The cache's rows follow the order of idx, in which two scores a rounding apart may change places: here the cache
    # comes back as what the token reads from it (an order-free sum over all its rows); "compact" returns the rows.
    return {"scores": comp.scores, "idx": comp.idx, "counts": comp.counts, "budgets": comp.budgets_all,
            "hits": comp.hits_all, "out": state["out"], "lse": state["lse_out"]}


def work(case):
    cfg = _cfg(case)
    elt = 2 if cfg.dtype == "bf16" else 4
    T, L, row = cfg.total_tokens, cfg.L, cfg.d * elt
    kept = sum(min(cfg.w, S) + min(cfg.mean_budget, S - cfg.w, cfg.layer_max) for S in cfg.seqlens) * L * cfg.Hkv
    scores, idx = 4 * L * cfg.Hkv * T, 4 * L * cfg.n_seqs * cfg.Hkv * cfg.layer_max
    token = 2 * L * cfg.n_seqs * cfg.Hq * (row + 4 * cfg.d)
    decode_flops = 4 * kept * cfg.d * cfg.G
    if case["what"] == "decode":
        return {"bytes": 2 * kept * row + token, "flops": decode_flops}
    if case["what"] == "compact":
        return {"bytes": scores + idx + 6 * kept * row, "flops": 0}      # rows to the cache, and from it to the packed copy
    q = L * cfg.n_seqs * cfg.Hq * cfg.w * row
    return {"bytes": L * cfg.Hkv * T * row + q + scores + idx + 4 * kept * row + token,
            "flops": 2 * L * cfg.Hq * cfg.w * T * cfg.d + decode_flops}


def tolerance(case):
    """Measured against the same cases with the scores in float64 (rounded once to fp32) and the decoding in float64.

    Scores differ by at most 4.1e-7 (2-norm) and 1.5e-6 (one value); 2e-4 of the index list change places (scores a
    rounding apart) and up to 1e-3 of the hit counts change by one. The decoding alone is off by 1.9e-6 and 2.1e-5. In a
    whole pass the budget line can fall between two scores a rounding apart: a KV head then keeps another row, of weight
    1 / 100 to 1 / 600, which takes its outputs off by up to half their size and the whole by up to 4e-3."""
    if case["what"] == "compact":
        return "exact"
    if case["what"] == "decode":
        return {"rel": 8e-6, "max": 8e-5}
    return {"rel": 4e-3, "max": 0.5, "differ": 4e-3}
