"""Timed cases of the adapter cache and the batched LoRA apply: what one serving iteration hands to the library.

A case is a dict of plain values.  Its fields:
  call      how the library is called: "one" (lora_apply: index and apply in one call), "each" (a plan per pass, then
            lora_apply_plan per projection), "all" (a plan per pass, then one lora_apply_plan_multi for every layer's
            projections), "linear" (a plan per pass, then lora_linear_plan per projection), "load" (whole adapters from
            pinned host memory, lora_cache_fill_slot_parts)
  projs     "q", "qkv", "qkvo" or "layer" (q, k, v, o, gate, up, down) of a model `hidden` wide with `inter` in its MLP
  layers    layer copies of the pool; a pass works on each once
  decode, prompts, plain   one-token requests; prompt lengths ("77,300", or "8x": eight drawn lognormally); one-token
            requests without an adapter
  pool, ranks, zipf, within_rank, distinct   adapters in the pool, the ranks they are drawn from, the exponent of their
            popularity (0: uniform), whether it runs within each rank, whether prompts have an adapter each
  batch     seed of the batch's structure (the values come from prepare()'s seed)
"""
import math

import numpy as np
import torch

from paper_2411_17741_amd import binding as B
from paper_2411_17741_amd.harness import CLASS_RANKS, slot_layout
from paper_2411_17741_amd.pool import LoraPool

SCALE = 2.0
FIVE = "8,16,32,64,128"  # the five adapter ranks of the configurations


def _case(name, call, projs, hidden, inter, layers, **kw):
    c = dict(name=name, call=call, dtype="bf16", projs=projs, hidden=hidden, inter=inter, layers=layers, decode=0, prompts="", plain=0,
             pool=100, ranks=FIVE, zipf=1.0, within_rank=False, distinct=False, direct=False, batch=1)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call there is: the full-precision configuration, 16 tokens in segments of 1, 3, 5 and 7
        _case("tiny_f32", "one", "q", 256, 256, 1, dtype="f32", prompts="1,3,5,7", pool=4, ranks="4,8,16", distinct=True),
        # one user, one token: every projection of a 7B model, launches and latency only
        _case("decode_one", "all", "layer", 4096, 11008, 32, decode=1, pool=8, ranks="16"),
        # an ordinary decode iteration: 64 requests over 100 adapters, q_proj of 32 layers
        _case("decode_64", "all", "q", 4096, 11008, 32, decode=64),
        # a loaded server: 512 requests over the paper's population of 200 adapters on the paper's four projections
        _case("decode_512_qkvo", "all", "qkvo", 4096, 11008, 8, decode=512, pool=200, within_rank=True),
        # one short prompt of odd length, called projection by projection as a model's forward pass does
        _case("prompt_short", "each", "layer", 4096, 11008, 4, prompts="77", pool=8, ranks="32"),
        # a prefill batch: eight prompts, an adapter each
        _case("prefill_8", "all", "q", 4096, 11008, 8, prompts="8x", ranks="16,64,128", zipf=0.0, distinct=True),
        # the large mixed batch: 224 decode requests beside 32 prompts, the full 7B layer, 500 adapters
        _case("mixed_7b", "all", "layer", 4096, 11008, 2, decode=224, prompts="32x", pool=500, zipf=1.2, batch=3),
        # a 13B layer: 512 decode requests beside four prompts of 512 tokens, 1000 adapters, some requests without one
        _case("stress_13b", "all", "layer", 5120, 13824, 2, decode=496, prompts="512,512,512,512", plain=16, pool=1000, zipf=1.2),
        # base projection and adapters in one pass: the prefill batch
        _case("linear_prefill", "linear", "q", 4096, 11008, 4, prompts="8x", ranks="16,64,128", zipf=0.0, distinct=True),
        # the same for a whole 13B layer with decode requests in the batch
        _case("linear_13b", "linear", "layer", 5120, 13824, 1, decode=496, prompts="512,512,512,512", plain=16, pool=1000, zipf=1.2),
        # adapters missing from the cache, one of each rank on q, k, v, o of 32 layers, through the staging buffers
        _case("load_staged", "load", "qkvo", 4096, 11008, 32, pool=5),
        # the same with pinned host memory read by the repacking kernel itself, all projections of eight layers
        _case("load_direct", "load", "layer", 4096, 11008, 8, pool=5, direct=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 4 + ["prompt"] * 3 + ["mixed"] * 2 + ["linear"] * 3 + ["load"] * 2 + ["f32"])
    hidden = 64 * rng.choice([16, 17, 24, 32, 40, 51, 64, 64, 64, 80])
    inter = 64 * int(round(hidden * 2.7 / 64))
    ranks = rng.choice([FIVE, FIVE, "16", "64", "4,12,24,48,96", "8,16", "32,128", "5,9,33,100"])
    kw = dict(ranks=ranks, zipf=rng.choice([0.0, 1.0, 1.2]), batch=rng.randrange(1, 1 << 20), pool=_log(rng, 4, 500))
    if kind == "decode":
        projs = rng.choice(["q", "qkv", "qkvo", "layer"])
        kw.update(decode=_log(rng, 1, 1024), plain=rng.choice([0, 0, 1, 9]))
        return _case("", rng.choice(["all", "all", "all", "each", "one"]), projs, hidden, inter, rng.choice([4, 8]), **kw)
    if kind == "prompt":
        lens = ",".join(str(_log(rng, 8, 2048)) for _ in range(rng.choice([1, 1, 2, 4, 8])))
        kw.update(prompts=lens, distinct=rng.random() < 0.5, pool=max(8, kw["pool"]))
        return _case("", rng.choice(["all", "all", "each"]), rng.choice(["q", "qkvo", "layer"]), hidden, inter, 2, **kw)
    if kind == "mixed":
        lens = ",".join(str(_log(rng, 16, 2048)) for _ in range(rng.randrange(1, 17)))
        kw.update(prompts=lens, decode=_log(rng, 8, 512), plain=rng.choice([0, 3, 40]))
        return _case("", "all", rng.choice(["qkvo", "layer"]), hidden, inter, 1, **kw)
    if kind == "linear":
        lens = ",".join(str(_log(rng, 64, 1024)) for _ in range(rng.choice([1, 2, 4])))
        kw.update(prompts=lens, decode=rng.choice([0, 0, 33, 200]), plain=rng.choice([0, 0, 5]))
        return _case("", "linear", rng.choice(["q", "qkvo"]), hidden, inter, 1, **kw)
    if kind == "load":
        kw.update(pool=rng.choice([1, 2, 3]), direct=rng.random() < 0.5)
        return _case("", "load", rng.choice(["qkvo", "layer"]), hidden, inter, rng.choice([4, 8]), **kw)
    kw.update(decode=_log(rng, 1, 64), pool=min(kw["pool"], 40), prompts=rng.choice(["", "5", "3,30"]))
    return _case("", rng.choice(["one", "all"]), rng.choice(["q", "qkv"]), rng.choice([256, 512, 1024]), 1024, 2, dtype="f32", **kw)


def _projs(case):
    """[(h_in, h_out, which activation tensor it reads)]"""
    h, i = case["hidden"], case["inter"]
    every = [(h, h, 0), (h, h, 0), (h, h, 0), (h, h, 1), (h, i, 2), (h, i, 2), (i, h, 3)]
    return every[: {"q": 1, "qkv": 3, "qkvo": 4, "layer": 7}[case["projs"]]]


def _batch(case):
    """The batch's structure: segment offsets, pool adapter (-1: none) and rank per segment, and the pool's ranks."""
    rng = np.random.default_rng(case["batch"])
    choices = [int(r) for r in case["ranks"].split(",")]
    n = case["pool"]
    if case["call"] == "load":
        return None, None, None, np.asarray([choices[a % len(choices)] for a in range(n)], np.int32)
    if case["prompts"].endswith("x"):  # a count
        lens = np.clip(np.rint(np.exp(rng.normal(6.0, 0.8, int(case["prompts"][:-1])))), 32, 2048).astype(np.int32)
    else:
        lens = np.asarray([int(v) for v in case["prompts"].split(",") if v], np.int32)
    n_req = case["decode"] + len(lens)
    perm = rng.permutation(n)  # popularity rank -> adapter
    per = n // len(choices) if case["within_rank"] else n
    p = np.arange(1, per + 1, dtype=np.float64) ** -case["zipf"]
    k = rng.choice(per, n_req, p=p / p.sum())
    if case["within_rank"]:  # as many adapters of every rank, the rank drawn first
        ranks = np.empty(n, np.int32)
        ranks[perm] = choices[-1]
        ranks[perm[: per * len(choices)]] = np.repeat(choices, per)
        pick = perm[rng.integers(0, len(choices), n_req) * per + k]
    else:
        ranks = rng.choice(choices, n).astype(np.int32)
        pick = perm[k]
    if case["distinct"] and len(lens):
        pick[case["decode"] :] = perm[np.arange(len(lens)) % n]
    lens = np.concatenate([np.ones(case["decode"], np.int32), lens, np.ones(case["plain"], np.int32)])
    pick = np.concatenate([pick, np.full(case["plain"], -1)])
    order = rng.permutation(len(lens))
    lens, pick = lens[order], pick[order].astype(np.int32)
    offsets = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return offsets, pick, np.where(pick >= 0, ranks[np.maximum(pick, 0)], 0).astype(np.int32), ranks


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    offsets, pick, seg_rank, ranks = _batch(case)
    projs, layers, load = _projs(case), case["layers"], case["call"] == "load"
    dtype = B.LORA_BF16 if case["dtype"] == "bf16" else B.LORA_F32
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    T = 1 if load else int(offsets[-1])

    def normal(*shape, sigma=1.0):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=dt).mul_(sigma)

    class_slots, slot_of = slot_layout(ranks)
    pool = LoraPool([p[:2] for p in projs], layers, CLASS_RANKS, class_slots, dtype, max_tokens=T,
                    max_segments=1 if load else len(pick), flags=B.LORA_CACHE_DIRECT_FILL if case["direct"] else 0)
    state = {"case": case, "pool": pool, "projs": projs}
    # adapter weights in pinned host memory.  Adapters that are loaded again in every pass have memory of their own; those that
    # are only in the pool share one piece of it, every part starting at another place
    used = np.arange(len(ranks)) if load else np.unique(pick[pick >= 0])
    sizes = [(int(ranks[a]) * h_in, int(ranks[a]) * h_out) for a in used for _ in range(layers) for h_in, h_out, _x in projs]
    total = sum(a + b for a, b in sizes) if load else (16 << 20) + max((max(s) for s in sizes), default=0)
    host = torch.empty(total, dtype=dt, pin_memory=True)
    for at in range(0, total, 64 << 20):
        host[at : at + (64 << 20)].copy_(normal(min(64 << 20, total - at), sigma=0.02))
    rng, at, i, jobs = np.random.default_rng(seed), 0, 0, []
    for a in used:
        parts = []
        for layer in range(layers):
            for p in range(len(projs)):
                na, nb = sizes[i]
                i += 1
                oa, ob = (at, at + na) if load else (int(v) * 64 for v in rng.integers(0, (16 << 20) // 64, 2))
                at += na + nb
                parts.append((layer, p, host.data_ptr() + oa * host.element_size(), host.data_ptr() + ob * host.element_size()))
        jobs.append((int(slot_of[a]), int(a) + 1, int(ranks[a]), B.make_fill_parts(parts)))
    if load:
        state.update(jobs=jobs, host=host, out=_slabs(pool, projs, layers, slot_of, ranks))
        return state
    stream = torch.cuda.current_stream().cuda_stream
    for slot, adapter, rank, parts in jobs:
        B.check(B.lora_cache_fill_slot_parts(pool.handle, slot, adapter, rank, 1.0, parts, stream))
    torch.cuda.synchronize()
    state["segs"] = (offsets, np.where(pick >= 0, slot_of[np.maximum(pick, 0)], -1).astype(np.int32), seg_rank)
    # activations: a set for every layer where only one projection is worked on, else shared by the layers; outputs of their own
    n_x = layers if len(projs) == 1 else 1
    state["x"] = [{k: normal(T, h_in) for h_in, _o, k in projs} for _ in range(n_x)]
    state["y"] = [normal(layers, T, h_out, sigma=1.28) for _i, h_out, _x in projs]
    if case["call"] == "linear":
        state["w"] = [[normal(h_out, h_in, sigma=0.02) for h_in, h_out, _x in projs] for _ in range(layers)]
        state["space"] = torch.empty(T * max(h_out for _i, h_out, _x in projs), dtype=torch.float32, device="cuda")
    if case["call"] == "all":
        state["descs"] = B.make_descs([(layer, p, state["x"][layer % n_x][projs[p][2]].data_ptr(), state["y"][p][layer].data_ptr())
                                       for layer in range(layers) for p in range(len(projs))])
    return state


def _slabs(pool, projs, layers, slot_of, ranks):
    """Per adapter, the bytes its slot holds: a view of the pool per projection and layer stride."""
    base, out = pool.buf.data_ptr(), []
    for a, slot in enumerate(slot_of):
        rows = (int(ranks[a]) + 7) // 8 * 8
        for p, (h_in, h_out, _x) in enumerate(projs):
            at = [B.lora_cache_slab(pool.handle, layer, p, int(slot))[1] - base for layer in range(2 if layers > 1 else 1)]
            n = rows * (h_in + h_out) * (2 if pool.dtype == B.LORA_BF16 else 4)
            out.append(torch.as_strided(pool.buf, (layers, n), (at[-1] - at[0] if layers > 1 else n, 1), at[0]))
    return out


def run(state):
    case, pool, projs = state["case"], state["pool"], state["projs"]
    stream = torch.cuda.current_stream().cuda_stream
    if case["call"] == "load":
        for slot, adapter, rank, parts in state["jobs"]:
            B.check(B.lora_cache_release_slot(pool.handle, slot))
            B.check(B.lora_cache_fill_slot_parts(pool.handle, slot, adapter, rank, 1.0, parts, stream))
        return state["out"]
    x, y = state["x"], state["y"]
    if case["call"] == "one":
        for layer in range(case["layers"]):
            for p, (_i, _o, k) in enumerate(projs):
                pool.apply(layer, p, x[layer % len(x)][k], y[p][layer], *state["segs"], SCALE)
        return y
    plan = pool.plan(x[0][0].shape[0], *state["segs"])
    if case["call"] == "all":
        B.check(B.lora_apply_plan_multi(pool.handle, plan, state["descs"], SCALE, stream))
    else:
        for layer in range(case["layers"]):
            for p, (_i, _o, k) in enumerate(projs):
                if case["call"] == "each":
                    pool.apply_plan(plan, layer, p, x[layer % len(x)][k], y[p][layer], SCALE)
                else:
                    B.check(B.lora_linear_plan(pool.handle, plan, layer, p, x[layer % len(x)][k].data_ptr(), state["w"][layer][p].data_ptr(),
                                               y[p][layer].data_ptr(), SCALE, stream, state["space"].data_ptr(), state["space"].numel() * 4))
    pool.plan_destroy(plan)
    return y


def work(case):
    offsets, pick, _r, ranks = _batch(case)
    projs, layers = _projs(case), case["layers"]
    e = 2 if case["dtype"] == "bf16" else 4
    if case["call"] == "load":  # every byte read from the host and written to the pool
        n = layers * sum(int(r) * (h_in + h_out) * e for r in ranks for h_in, h_out, _x in projs)
        return {"bytes": 2 * n, "flops": 0}
    tokens = np.where(pick >= 0, np.diff(offsets), 0)
    T, n, weights = int(offsets[-1]), int(tokens.sum()), int(ranks[np.unique(pick[pick >= 0])].sum())
    token_ranks = int((tokens * np.where(pick >= 0, ranks[np.maximum(pick, 0)], 0)).sum())
    linear = case["call"] == "linear"
    rows = T if linear else n
    n_bytes = sum(rows * h_in * e for h_in in {k: h for h, _o, k in projs}.values())  # activations once per group that shares them
    flops = 0
    for h_in, h_out, _x in projs:
        n_bytes += weights * (h_in + h_out) * e
        flops += 2 * token_ranks * (h_in + h_out)
        if linear:
            n_bytes += T * h_out * e + h_in * h_out * e
            flops += 2 * T * h_in * h_out
        else:
            n_bytes += 2 * n * h_out * e
    return {"bytes": layers * n_bytes, "flops": layers * flops}


def tolerance(case):
    if case["call"] == "load":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 2e-7, "max": 1e-6}  # four times what one pass differs from itself in 64 bits by; bf16 the same
    return {"rel": 7e-3, "max": 3e-2}
