"""Lists of GEMV work with more projections or super-chunks than 120 and 768: one launch of up to 224 and 1536 where they are of at most eight kinds, several launches otherwise.
Every entry against a call of its own."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SEVEN = [(256, 256)] * 3 + [(256, 128), (256, 1088), (256, 64), (1088, 256)]  # 0..5 read one x
WIDE = [(64, 9216), (64, 6144)]  # 9 and 6 super-chunks
CASES = {  # projections, layers, requests per slot, ranks
    "121 entries": (SEVEN[:1], 121, [1], [16]),
    "224 entries": (SEVEN, 32, [1], [16]),
    "225 entries": (SEVEN[:1], 225, [1], [8]),
    "231 entries": (SEVEN, 33, [1, 1, 3], [16, 128, 40]),
    "wide items": (SEVEN, 32, [9, 17, 4, 1, 2], [128, 16, 33, 8, 64]),
    "super-chunks": (WIDE, 70, [1], [32]),                      # 1050 in 140 entries
    "more super-chunks than a launch": (WIDE, 112, [2, 1], [8, 16]),  # 1680 in 224
    "super-chunks of few entries": (WIDE, 55, [1], [16]),       # 825 in 110
    "eight kinds": (SEVEN + [(256, 320)], 28, [1], [16]),
    "nine kinds": (SEVEN + [(256, 320), (256, 384)], 25, [1], [16]),
    "requests for fewer sets": (SEVEN, 32, [120, 150, 80], [16, 8, 32]),
}

# GEMV launches of a list: those of more than 224 entries or 1536 super-chunks take another, those of nine kinds run in batches of 120, and so do those of tokens for which there
# are no more sets; a list of 225 leaves one entry over
LAUNCHES = {case: 1 for case in CASES}
LAUNCHES |= {"225 entries": 2, "231 entries": 2, "more super-chunks than a launch": 2, "requests for fewer sets": 2, "nine kinds": 3}


def _setup(case, dtype, flags):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    projs, layers, counts, ranks = CASES[case]
    slot = np.random.default_rng(1).permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)
    T, bf16 = len(slot), dtype == "bf16"
    dt = torch.bfloat16 if bf16 else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(layers)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda", dtype=dt).mul_(sigma)
    pool = LoraPool(projs, layers, [128], [len(ranks)], B.LORA_BF16 if bf16 else B.LORA_F32, max_tokens=T, max_segments=T, mfma_min_tokens=1000 if bf16 else 0,
                    flags=B.LORA_CACHE_SPLIT_GEMV if flags == "split" else 0)
    for s, r in enumerate(ranks):
        for layer in range(layers):
            for p, (h_in, h_out) in enumerate(projs):
                pool.fill(s, s + 1, r, 0.5 + s, layer, p, normal(h_in, r, sigma=0.05).cpu(), normal(r, h_out, sigma=0.05).cpu())
    torch.cuda.synchronize()
    plan = pool.plan(T, np.arange(T + 1, dtype=np.int32), slot, np.asarray(ranks, np.int32)[slot])
    xs = {h: normal(T, h) for h in {h for h, _o in projs}}
    entries = [(layer, p) for layer in range(layers) for p in range(len(projs))]
    base = [normal(T, projs[p][1]) for _l, p in entries]
    want = [y.clone() for y in base]
    for (layer, p), y in zip(entries, want):
        pool.apply_plan(plan, layer, p, xs[projs[p][0]], y, 2.0)
    torch.cuda.synchronize()
    y = [t.clone() for t in base]
    descs = B.make_descs([(layer, p, xs[projs[p][0]].data_ptr(), t.data_ptr()) for (layer, p), t in zip(entries, y)])
    return B, pool, plan, descs, base, want, y, xs


def _check(got, want, dtype):
    # wide items and single ones split their sums in other places: see the bound of the batches' test
    rel = floor = 2.0**-7 if dtype == "bf16" else 2.0**-20
    for k, (g, w) in enumerate(zip(got, want)):
        g, w = g.double(), w.double()
        err, rms = (g - w).abs(), w.pow(2).mean().sqrt()
        assert bool((err <= rel * w.abs() + floor * rms).all()), f"entry {k}: {float((err / rms).max())}"


@pytest.mark.parametrize("dtype,flags,case", [(d, "auto", c) for d in ("bf16", "f32") for c in CASES] + [("bf16", "split", c) for c in ("224 entries", "wide items")])
def test_lists_against_single_calls(case, dtype, flags):
    B, pool, plan, descs, _base, want, y, _xs = _setup(case, dtype, flags)
    try:
        B.lora_cache_set_timing(pool.handle, 1)
        B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        pool.check_fault()
        rc, t = B.lora_cache_read_timing(pool.handle)
        assert rc == B.LORA_OK
        assert {k: n for k, (_ms, n) in t.items() if n} == {k: LAUNCHES[case] for k in (["gemv_shrink", "gemv_expand"] if flags == "split" else ["gemv_fused"])}
        _check(y, want, dtype)
    finally:
        pool.close()


@pytest.mark.parametrize("case", ["224 entries", "wide items"])
def test_a_captured_list_replays(case):
    B, pool, plan, descs, base, want, y, _xs = _setup(case, "bf16", "auto")
    try:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
        for i in range(3):
            for t, b in zip(y, base):
                t.copy_(b)
            graph.replay()
            torch.cuda.synchronize()
            pool.check_fault()
            _check(y, want, "bf16")
            if i == 1:  # eager work in between
                B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
    finally:
        pool.close()
