"""Performance cases of the relay-race ranking path: what a serving instance has this library do.

Three calls make up the path: `prefill` (relaygr_prefill_prefix: pre-inference that leaves a user's per-layer
K/V in the HBM pool), `rank` (relaygr_rank_with_cache: score candidates against cached prefixes, recomputing the
users that have none) and `full` (relaygr_rank_full_recompute: inference without a cache).  A case names the call,
the model (layers, width, heads, storage type, attention form) and the jagged batch:

    users                  users in the call
    prefix, prefix_sigma   prefix tokens per user: all `prefix` (sigma 0), or lognormal around it with that sigma,
                           clipped to [prefix_min, prefix_max]
    cands_lo, cands_hi     candidates per user, uniform in the range
    suffix_lo, suffix_hi   short-term suffix tokens per user, uniform in the range
    miss_tenths            of ten users, how many have no cached prefix when they are ranked
    shape_seed             seed of those lengths, which belong to the case; the values belong to prepare()'s seed

Weights, biases and LayerNorm offsets are N(0, 0.02^2), LayerNorm gains 1 + N(0, 0.02^2) and embeddings
N(0, 0.02^2), as in the workloads of synth/generator.py, whose model shapes and length recipes are used throughout.
"""
import math
import random

import numpy as np
import torch

import paper_2601_01712_amd as rg
from synth.generator import ModelConfig

PAGE_TOKENS = 256       # tokens per pool page, as in the benchmark
_STD = 0.02
_TORCH = {"fp32": torch.float32, "bf16": torch.bfloat16, "fp16": torch.float16}


def _case(call, layers, d, heads, dtype, users, prefix, cands, suffix=(0, 0), attention="silu", prefix_sigma=0.0, miss_tenths=0, shape_seed=0):
    return {"call": call, "layers": layers, "d": d, "heads": heads, "dtype": dtype, "attention": attention, "users": users,
            "prefix": prefix, "prefix_sigma": prefix_sigma, "prefix_min": min(512, prefix), "prefix_max": 16384,
            "cands_lo": cands[0], "cands_hi": cands[1], "suffix_lo": suffix[0], "suffix_hi": suffix[1],
            "miss_tenths": miss_tenths, "shape_seed": shape_seed}


def listed():
    cases = {
        # the smallest model and request: launches and host work are all there is
        "rank_tiny_fp32": _case("rank", 2, 64, 2, "fp32", 1, 256, (16, 16)),
        # one request of the storage type and model the paper's cache sizes are quoted in (8 layers, width 256, 2K tokens)
        "rank_fp32": _case("rank", 8, 256, 4, "fp32", 1, 2048, (512, 512)),
        # one request by itself: the latency a user waits for
        "rank_one_user": _case("rank", 8, 512, 8, "bf16", 1, 4096, (512, 512)),
        # a small model under a small batch, with short-term suffixes
        "rank_small_model": _case("rank", 4, 256, 4, "bf16", 8, 2048, (256, 256), suffix=(16, 16)),
        # the batch the throughput is quoted on
        "rank_batch": _case("rank", 8, 512, 8, "bf16", 16, 4096, (512, 512)),
        # long histories, many candidates
        "rank_long": _case("rank", 8, 512, 8, "bf16", 32, 8192, (1000, 1000)),
        # production-shaped: ragged lengths throughout, three users in ten without a cached prefix (the largest case)
        "rank_jagged_misses": _case("rank", 8, 512, 8, "bf16", 64, 4096, (200, 2000), suffix=(0, 64), prefix_sigma=0.7, miss_tenths=3, shape_seed=5),
        # the wide end of the embedding axis
        "rank_wide": _case("rank", 8, 1024, 8, "bf16", 16, 4096, (512, 512)),
        # the second attention form on a ragged batch of cached users
        "rank_softmax": _case("rank", 8, 512, 8, "bf16", 16, 4096, (200, 2000), suffix=(0, 64), attention="softmax", prefix_sigma=0.7, shape_seed=9),
        # pre-inference as it is issued, one user at a time as they arrive
        "prefill_one_user": _case("prefill", 8, 512, 8, "bf16", 1, 4099, (0, 0)),
        # pre-inference of a ragged batch, in half precision
        "prefill_batch_fp16": _case("prefill", 8, 512, 8, "fp16", 16, 4096, (0, 0), prefix_sigma=0.7, shape_seed=8),
        # one request that found no cached prefix
        "full_one_user": _case("full", 8, 512, 8, "bf16", 1, 4096, (512, 512), suffix=(21, 21)),
    }
    return [dict(c, name=name) for name, c in cases.items()]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        call = rng.choice(["rank", "rank", "rank", "prefill", "full"])
        shape_seed = rng.randrange(1 << 20)
        family = rng.random()
        if family < 0.15:       # the tiny fp32 model
            case = _case(call, 2, 64, 2, "fp32", rng.randint(1, 4), _log_int(rng, 16, 2048), (_log_int(rng, 1, 256),) * 2,
                         suffix=(rng.randint(0, 20),) * 2, shape_seed=shape_seed)
        elif family < 0.3:      # the paper's fp32 model
            case = _case(call, 8, 256, 4, "fp32", rng.randint(1, 3), _log_int(rng, 256, 4096), (_log_int(rng, 32, 1000),) * 2,
                         suffix=(rng.randint(0, 64),) * 2, shape_seed=shape_seed)
        else:                   # the 16-bit models, one user to a full batch
            layers, d, heads = rng.choice([(4, 256, 4), (8, 512, 8), (8, 512, 8), (8, 512, 8), (8, 1024, 8)])
            jagged = rng.random() < 0.5
            m = _log_int(rng, 32, 2048)
            case = _case(call, layers, d, heads, rng.choice(["bf16", "bf16", "bf16", "fp16"]), _log_int(rng, 1, 64), _log_int(rng, 512, 16384),
                         (max(1, m // 4), m) if jagged else (m, m), suffix=(0, rng.randint(0, 64)) if jagged else (rng.choice([0, 0, 16, 33]),) * 2,
                         attention=rng.choice(["silu", "silu", "silu", "softmax"]), prefix_sigma=0.7 if jagged else 0.0,
                         miss_tenths=rng.choice([0, 0, 3]), shape_seed=shape_seed)
        if case["call"] == "prefill":
            case.update(cands_lo=0, cands_hi=0, suffix_lo=0, suffix_hi=0)
        if case["call"] != "rank":
            case["miss_tenths"] = 0
        if _cost(case) <= most:
            return case


def _lengths(case):
    """Per-user prefix, suffix and candidate counts and whether the prefix is cached: a function of the case alone."""
    r = random.Random(case["shape_seed"])
    L, S, M, cached = [], [], [], []
    for _ in range(case["users"]):
        p = case["prefix"]
        if case["prefix_sigma"] > 0:
            p = min(case["prefix_max"], max(case["prefix_min"], int(round(math.exp(r.gauss(math.log(p), case["prefix_sigma"]))))))
        L.append(p)
        S.append(r.randint(case["suffix_lo"], case["suffix_hi"]))
        M.append(r.randint(case["cands_lo"], case["cands_hi"]))
        cached.append(case["call"] != "full" and r.randrange(10) >= case["miss_tenths"])
    return L, S, M, cached


def work(case):
    L, S, M, cached = _lengths(case)
    d, e, layers = case["d"], 4 if case["dtype"] == "fp32" else 2, case["layers"]
    prefill = case["call"] == "prefill"
    computed = sum(l for l, c in zip(L, cached) if prefill or not c)                    # prefix tokens run through the layers
    causal = sum(l * (l + 1) // 2 for l, c in zip(L, cached) if prefill or not c)       # and the keys they see
    new = sum(S) + sum(M)
    seen = sum(m * (l + s + 1) + s * l + s * (s + 1) // 2 for l, s, m in zip(L, S, M))  # keys suffix and candidate tokens see
    # projections 8 d^2 and 2 d^2 per token and layer; prefix tokens need only their K and V in the last layer
    flops = new * layers * 10 * d * d + computed * ((layers - 1) * 10 + 4) * d * d
    flops += 4 * d * (layers * seen + (layers - 1) * causal)
    weights = layers * (5 * d * d + 9 * d) + 3 * d
    cache = 2 * layers * d * sum(L) if prefill else 2 * layers * d * sum(l for l, c in zip(L, cached) if c)
    return {"bytes": e * (weights + cache + (computed + new) * d) + 4 * sum(M), "flops": flops}


def _cost(case):
    """Rough time of a pass, to keep drawn cases within the listed ones: 32-bit arithmetic has a small part of the rate."""
    w = work(case)
    return w["flops"] * (64 if case["dtype"] == "fp32" else 1) / 8e14 + w["bytes"] / 4e12


def tolerance(case):
    # Storage types of 8, 11 and 24 significant bits; activations are rounded to them several times a layer.  Against the
    # same model in float64 the scores of 8 layers are off by 8e-3, 1.1e-3 and 1e-6; two summation orders of one call
    # (prefixes cached and recomputed) differ by 4e-3, 8e-4 and 1.2e-6.
    return {"rel": {"bf16": 1e-2, "fp16": 2e-3, "fp32": 1e-5}[case["dtype"]]}


def _weights(model, gen):
    d = model.d_model

    def normal(*shape, mean=0.0):
        return (torch.randn(shape, generator=gen, device="cuda:0") * _STD + mean).cpu().numpy()

    layers = [{"ln_in_g": normal(d, mean=1.0), "ln_in_b": normal(d), "w1": normal(4 * d, d), "b1": normal(4 * d),
               "ln_at_g": normal(d, mean=1.0), "ln_at_b": normal(d), "w2": normal(d, d), "b2": normal(d)} for _ in range(model.n_layers)]
    return {"layers": layers, "ln_out_g": normal(d, mean=1.0), "ln_out_b": normal(d), "w_score": normal(d), "b_score": 0.01}


def _batch(case, users, lengths, gen, with_prefix):
    """The listed users of the case as a batch; `with_prefix`: whether their prefix embeddings are at hand."""
    L, S, M, _ = lengths

    def off(x):
        return np.concatenate([[0], np.cumsum([x[u] for u in users])]).astype(np.int32)

    def emb(rows):
        return (torch.randn((rows, case["d"]), generator=gen, device="cuda:0") * _STD).to(_TORCH[case["dtype"]])

    po, so, co = off(L), off(S), off(M)
    return rg.Batch({"n_users": len(users), "user_ids": np.asarray(users, dtype=np.uint64) + np.uint64(1000),
                     "prefix_emb": emb(int(po[-1]) if with_prefix else 0), "prefix_off": po,
                     "suffix_emb": emb(int(so[-1])), "suffix_off": so, "cand_emb": emb(int(co[-1])), "cand_off": co}, case["dtype"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    lengths = _lengths(case)
    L, S, M, cached = lengths
    n = case["users"]
    model = ModelConfig(case["layers"], case["d"], case["heads"], case["dtype"], attention=case["attention"])
    ctx = rg.Context(model, _weights(model, gen), n, sum(L), sum(S) + sum(M))
    batch = _batch(case, range(n), lengths, gen, with_prefix=case["call"] != "rank" or not all(cached))
    state = {"call": case["call"], "ctx": ctx, "pool": None, "batch": batch}
    if case["call"] != "full":
        hit = [u for u in range(n) if cached[u] or case["call"] == "prefill"]
        slab = sum(rg.relaygr_kv_pool_bytes_for(ctx.cfg, L[u], PAGE_TOKENS) for u in hit)
        pool = rg.KvPool(ctx.cfg, case["dtype"], max(slab, rg.relaygr_kv_pool_bytes_for(ctx.cfg, 1, PAGE_TOKENS)), PAGE_TOKENS)
        pool.slab.zero_()       # pages are whole: the tokens behind a prefix's last tile are never written
        handles = np.zeros(n, dtype=np.uint64)
        for u in hit:
            handles[u] = rg.relaygr_kv_pool_alloc(pool, 1000 + u, L[u])
        batch.set_handles(handles)
        if case["call"] == "rank" and hit:      # the cached users' prefixes have been pre-inferred some time ago
            pre = _batch(case, hit, (L, [0] * n, [0] * n, cached), gen, with_prefix=True)
            pre.set_handles(handles[hit])
            rg.relaygr_prefill_prefix(ctx, pool, pre)
            torch.cuda.synchronize()
        state["pool"] = pool
    if case["call"] != "prefill":
        state["scores"] = torch.empty(sum(M), dtype=torch.float32, device="cuda:0")
    return state


def run(state):
    if state["call"] == "prefill":
        rg.relaygr_prefill_prefix(state["ctx"], state["pool"], state["batch"])
        return state["pool"].elements()
    if state["call"] == "rank":
        return rg.relaygr_rank_with_cache(state["ctx"], state["pool"], state["batch"], state["scores"])
    return rg.relaygr_rank_full_recompute(state["ctx"], state["batch"], state["scores"])
