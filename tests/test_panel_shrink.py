"""The tile shrink by panels: how panels and projections fall to blocks (no GPU needed), and the results at the edges of panels, of their rank blocks and of the k slices."""
import numpy as np
import pytest
import torch

from paper_2411_17741_amd import binding as B

RANKS = [5, 16, 17, 33, 64, 65, 96, 97, 128, 8]  # the last and first ranks of every number of rank blocks


def _segments(lens, seed=0):
    """Segments in a drawn order; every slot has the rank RANKS[slot % 10]."""
    order = np.random.default_rng(seed).permutation(len(lens))
    lens = np.asarray(lens)[order]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    slot = order.astype(np.int32) % 20
    return off, slot, np.asarray(RANKS, np.int32)[slot % 10]


@pytest.mark.parametrize("lens", [[1] * 3 + [8], [192], [193, 64, 65], [40] * 20, [1000, 192, 191, 16, 129, 128, 700, 400, 33, 64] * 3, list(range(8, 700, 23))])
def test_every_row_once_per_projection(lens):
    off, slot, rank = _segments(lens)
    T = int(off[-1])
    cfg = B.make_config([(512, 256)], 1, [128], [20], B.LORA_BF16, T, len(lens), mfma_min_tokens=8, flags=B.LORA_CACHE_HOST_ONLY)
    rc, h = B.lora_cache_create(cfg, 0, 0)
    assert rc == B.LORA_OK
    for s in range(20):
        assert B.lora_cache_fill_slot(h, s, s + 1, RANKS[s % 10], 1.0 + s, 0, 0, 0, 0) == B.LORA_OK
    rc, plan = B.lora_plan_create(h, T, off, slot, rank)
    assert rc == B.LORA_OK
    rc, units, toks = B.lora_plan_dump(h, plan, 0)
    assert rc == B.LORA_OK
    in_tiles = np.zeros(T, np.int64)
    for u in units[units["kind"] == B.LORA_UNIT_TILE]:
        in_tiles[toks[u["tok_off"] : u["tok_off"] + u["n_tok"]]] += 1
    assert in_tiles.any()
    slot_of, rank_of = np.repeat(slot, np.diff(off)), np.repeat(rank, np.diff(off))
    panels = units[units["kind"] == B.LORA_UNIT_PANEL_SHRINK]
    for gn in range(1, 5):
        cover = np.zeros((gn, T), np.int64)
        for u in panels[panels["where"] == gn]:
            t = toks[u["tok_off"] : u["tok_off"] + u["n_tok"]]
            assert 1 <= u["n_tok"] <= 192 and 0 <= u["lo"] < u["hi"] <= gn and u["hi"] - u["lo"] <= 3
            assert (slot_of[t] == u["slot"]).all() and (rank_of[t] == u["rank"]).all() and u["alpha"] == 1.0 + u["slot"]
            blocks = next(n for n in (1, 2, 4, 6, 8) if 16 * n >= u["rank"])
            assert -(-u["n_tok"] // 64) * 64 + 16 * blocks * (u["hi"] - u["lo"]) <= 416  # a stage's rows: three stages fit into LDS
            cover[u["lo"] : u["hi"], t] += 1
        assert (cover == in_tiles).all()
    assert B.lora_plan_destroy(h, plan) == B.LORA_OK and B.lora_cache_destroy(h) == B.LORA_OK


# (widths of 1, 5 and 17 stages of 64 k: one slice; 40 and 129: several for the short lists)
@pytest.mark.gpu
@pytest.mark.parametrize("h_in", [64, 320, 1088, 2560, 8256])
@pytest.mark.parametrize("lens", [
    [2000, 1201, 833, 400, 385, 1409, 1, 1, 1] * 2 + [9, 24] * 3,  # panels of 129 to 192 rows; pools of one-token requests beside them
    [193, 65, 64, 63, 129, 1, 577, 192, 128, 191] * 12,        # pools of several segments; gathered panels
    [1] * 3000 + [300] * 30,                                   # gathered panels of many requests
])
def test_against_torch(lens, h_in):
    from paper_2411_17741_amd.pool import LoraPool

    off, slot, rank = _segments(lens, seed=h_in)
    T, h_out, groups = int(off[-1]), 64, [1, 3, 4, 2]  # four groups of projections that share their input
    n = sum(groups)
    gen = torch.Generator(device="cuda").manual_seed(h_in)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    x = [normal(T, h_in) for _ in groups]
    x_of = [g for g, k in enumerate(groups) for _ in range(k)]
    A = [[normal(h_in, RANKS[s % 10], sigma=0.02) for s in range(20)] for _ in range(n)]
    Bm = [normal(RANKS[s % 10], h_out, sigma=0.02) for s in range(20)]
    slot_of_token = torch.as_tensor(np.repeat(slot, np.diff(off)), device="cuda")
    pool = LoraPool([(h_in, h_out)] * n, 1, [128], [20], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=8)
    try:
        pool.buf.fill_(0xFF)  # NaN in every word that is not written: the next pool takes the same memory
        pool.close()
        pool = LoraPool([(h_in, h_out)] * n, 1, [128], [20], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=8)
        for s in range(20):
            for p in range(n):
                pool.fill(s, s + 1, RANKS[s % 10], 0.5 + s / 8, 0, p, A[p][s].cpu(), Bm[s].cpu())
        plan = pool.plan(T, off, slot, rank)
        base = normal(n, T, h_out)
        for entries in (range(n), range(1, 4), [0], [4, 5, 6, 7]):  # a batch of all, and single groups
            y = base.clone()
            descs = B.make_descs([(0, p, x[x_of[p]].data_ptr(), y[p].data_ptr()) for p in entries])
            B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
            pool.check_fault()
            for p in entries:
                ref, rounding = base[p].double(), torch.zeros(T, h_out, dtype=torch.float64, device="cuda")
                for s in range(20):
                    at = slot_of_token == s
                    v = 2.0 * (0.5 + s / 8) * (x[x_of[p]][at].double() @ A[p][s].double())
                    ref[at] += v @ Bm[s].double()
                    rounding[at] = v.abs() @ Bm[s].double().abs()
                # the rounding of the output (2^-8 of its value) and that of every entry of s.v (2^-8 of its term); an eighth more for the sums in fp32
                assert bool(((y[p].double() - ref).abs() <= 1.125 * 2.0**-8 * (ref.abs() + rounding)).all()), (p, list(entries))
            for p in set(range(n)) - set(entries):
                assert torch.equal(y[p], base[p])
    finally:
        pool.close()


# Crossed: a slot for every length and rank.  A block's body is one of (runs of 64 rows, rank blocks, projections), in one slice or in several
CROSS_RANKS = RANKS + [32, 80]
CROSS = [  # lengths, width, more than one slice
    ([9, 63, 64, 65, 100, 128, 129, 191, 192], 64, False),
    ([9, 63, 64, 65, 100, 128, 129, 191, 192], 320, False),
    ([9, 63, 65, 129, 191], 2560, True),
    ([64, 128, 192], 4160, True),
    ([33, 100, 177], 8256, True),
]


def _crossed(lens):
    pairs = [(n, r) for n in lens for r in CROSS_RANKS]
    order = np.random.default_rng(len(lens)).permutation(len(pairs))
    off = np.concatenate([[0], np.cumsum([pairs[i][0] for i in order])]).astype(np.int32)
    return off, order.astype(np.int32), np.asarray([r for _n, r in pairs], np.int32)


def _check_bodies(handle, plan, sliced):
    """Launches for 1 to 4 projections that read the same x run by panels, and between them reach every body."""
    rc, units, _toks = B.lora_plan_dump(handle, plan, 0)
    assert rc == B.LORA_OK
    ways = units[units["kind"] == B.LORA_UNIT_SHRINK_WAY]
    assert list(ways["where"]) == [1, 2, 3, 4]
    reached = set()
    for w in ways:
        if w["lo"] == 2 and (w["hi"] > 1) == sliced:
            for u in units[(units["kind"] == B.LORA_UNIT_PANEL_SHRINK) & (units["where"] == w["where"])]:
                reached.add((-(-int(u["n_tok"]) // 64), next(n for n in (1, 2, 4, 6, 8) if 16 * n >= u["rank"]), int(u["hi"] - u["lo"])))
    every = {(runs, nb, n) for runs in (1, 2, 3) for nb in (1, 2, 4, 6, 8) for n in range(1, min(3, (416 - 64 * runs) // (16 * nb)) + 1)}
    assert reached == every, every - reached


@pytest.mark.parametrize("lens,h_in,sliced", CROSS)
def test_every_body_is_reached(lens, h_in, sliced):
    off, slot, ranks = _crossed(lens)
    cfg = B.make_config([(h_in, 64)] * 4, 1, [128], [len(ranks)], B.LORA_BF16, int(off[-1]), len(slot), mfma_min_tokens=8, flags=B.LORA_CACHE_HOST_ONLY)
    rc, h = B.lora_cache_create(cfg, 0, 0)
    assert rc == B.LORA_OK
    for s, r in enumerate(ranks):
        assert all(B.lora_cache_fill_slot(h, s, s + 1, int(r), 1.0, 0, p, 0, 0) == B.LORA_OK for p in range(4))
    rc, plan = B.lora_plan_create(h, int(off[-1]), off, slot, ranks[slot])
    assert rc == B.LORA_OK
    _check_bodies(h, plan, sliced)  # (of 256 compute units)
    assert B.lora_plan_destroy(h, plan) == B.LORA_OK and B.lora_cache_destroy(h) == B.LORA_OK


@pytest.mark.gpu
@pytest.mark.parametrize("lens,h_in,sliced", CROSS)
def test_every_body_against_torch(lens, h_in, sliced):
    from paper_2411_17741_amd.pool import LoraPool

    off, slot, ranks = _crossed(lens)
    T, h_out, n = int(off[-1]), 64, len(ranks)
    gen = torch.Generator(device="cuda").manual_seed(h_in)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    x = normal(T, h_in)
    A = [[normal(h_in, r, sigma=0.02) for r in CROSS_RANKS] for _ in range(4)]
    Bm = [normal(r, h_out, sigma=0.02) for r in CROSS_RANKS]
    host_a, host_b = [[a.cpu().pin_memory() for a in row] for row in A], [b.cpu().pin_memory() for b in Bm]
    make = lambda: LoraPool([(h_in, h_out)] * 4, 1, [128], [n], B.LORA_BF16, max_tokens=T, max_segments=n, mfma_min_tokens=8)
    pool = make()
    try:
        pool.buf.fill_(0xFF)  # NaN in every word that is not written: the next pool takes the same memory
        pool.close()
        pool = make()
        stream = torch.cuda.current_stream().cuda_stream
        for s in range(n):
            k = s % len(CROSS_RANKS)
            parts = B.make_fill_parts([(0, p, host_a[p][k].data_ptr(), host_b[k].data_ptr()) for p in range(4)])
            B.check(B.lora_cache_fill_slot_parts(pool.handle, s, s + 1, int(ranks[s]), 0.5 + s / 64, parts, stream))
        plan = pool.plan(T, off, slot, ranks[slot])
        if torch.cuda.get_device_properties(0).multi_processor_count == 256:
            _check_bodies(pool.handle, plan, sliced)
        base = normal(4, T, h_out)
        slot_of_token = torch.as_tensor(np.repeat(slot, np.diff(off)), device="cuda")
        factor = 2.0 * (0.5 + slot_of_token.double() / 64)
        ref, rounding = base.double(), torch.zeros(4, T, h_out, dtype=torch.float64, device="cuda")
        for p in range(4):
            for k in range(len(CROSS_RANKS)):
                at = slot_of_token % len(CROSS_RANKS) == k
                v = factor[at, None] * (x[at].double() @ A[p][k].double())
                ref[p, at] += v @ Bm[k].double()
                rounding[p, at] = v.abs() @ Bm[k].double().abs()
        for gn in range(1, 5):
            y = base.clone()
            B.check(B.lora_apply_plan_multi(pool.handle, plan, B.make_descs([(0, p, x.data_ptr(), y[p].data_ptr()) for p in range(gn)]), 2.0, stream))
            pool.check_fault()
            # the rounding of the output (2^-8 of its value) and that of every entry of s.v (2^-8 of its term); an eighth more for the sums in fp32
            assert bool(((y[:gn].double() - ref[:gn]).abs() <= 1.125 * 2.0**-8 * (ref[:gn].abs() + rounding[:gn])).all()), gn
            assert torch.equal(y[gn:], base[gn:])
    finally:
        pool.close()


@pytest.mark.gpu
@pytest.mark.parametrize("lens,ranks,by_table", [
    ([101, 101], [128, 128], [3, 4]),
    ([150, 149, 148, 149], [128] * 4, [1]),
    ([60, 59, 58, 57], [128, 120, 97, 128], [3, 4]),
])
def test_launches_that_the_run_table_takes(lens, ranks, by_table):
    """Long input rows and few tiles: neither the short launch's units nor panels; by_table: for how many projections that read the same x."""
    from paper_2411_17741_amd.pool import LoraPool

    h_in, h_out, T, n = 13824, 128, sum(lens), len(lens)
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    A, Bm = [[normal(h_in, r, sigma=0.01) for r in ranks] for _ in range(4)], [normal(r, h_out, sigma=0.02) for r in ranks]
    x, base = normal(T, h_in), normal(4, T, h_out)
    pool = LoraPool([(h_in, h_out)] * 4, 1, [128], [n], B.LORA_BF16, max_tokens=T, max_segments=n, mfma_min_tokens=8)
    try:
        for s in range(n):
            for p in range(4):
                pool.fill(s, s + 1, ranks[s], 0.5 + s, 0, p, A[p][s].cpu(), Bm[s].cpu())
        plan = pool.plan(T, off, np.arange(n, dtype=np.int32), np.asarray(ranks, np.int32))
        rc, units, _toks = B.lora_plan_dump(pool.handle, plan, 0)
        ways = units[units["kind"] == B.LORA_UNIT_SHRINK_WAY]
        assert rc == B.LORA_OK and (list(ways[ways["lo"] == 1]["where"]) == by_table or torch.cuda.get_device_properties(0).multi_processor_count != 256)
        for gn in by_table:
            y = base.clone()
            B.check(B.lora_apply_plan_multi(pool.handle, plan, B.make_descs([(0, p, x.data_ptr(), y[p].data_ptr()) for p in range(gn)]), 2.0, torch.cuda.current_stream().cuda_stream))
            pool.check_fault()
            for p in range(gn):
                for s in range(n):
                    a, b = int(off[s]), int(off[s + 1])
                    v = 2.0 * (0.5 + s) * (x[a:b].double() @ A[p][s].double())
                    ref, rounding = base[p, a:b].double() + v @ Bm[s].double(), v.abs() @ Bm[s].double().abs()
                    assert bool(((y[p, a:b].double() - ref).abs() <= 1.125 * 2.0**-8 * (ref.abs() + rounding)).all()), (gn, p, s)  # as above
    finally:
        pool.close()
