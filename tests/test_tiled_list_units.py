"""The lists with tiles that a plan holds besides its own, as list calls and the base product read them: which token takes which path with which entry (no GPU needed)."""
import numpy as np
import pytest

from paper_2411_17741_amd import binding as B
from plan_checks import check_plan_units

LAYER = [(1024, 1024)] * 4 + [(1024, 2752)] * 2 + [(2752, 1024)]


def _plan(lens, slot, ranks, projs, layers, dtype=B.LORA_BF16, **kw):
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    slot = np.asarray(slot, np.int32)
    rank = np.asarray([ranks[s] if s >= 0 else 0 for s in slot], np.int32)
    kw.setdefault("flags", B.LORA_CACHE_HOST_ONLY)
    rc, h = B.lora_cache_create(B.make_config(projs, layers, [128], [len(ranks)], dtype, int(off[-1]), len(lens), **kw), 0, 0)
    assert rc == B.LORA_OK
    for s, r in enumerate(ranks):
        for layer in range(layers):
            for p in range(len(projs)):
                assert B.lora_cache_fill_slot(h, s, 7 + s, r, 1.0 + s, layer, p, 0, 0) == B.LORA_OK
    rc, plan = B.lora_plan_create(h, int(off[-1]), off, slot, rank)
    assert rc == B.LORA_OK
    return h, plan, (int(off[-1]), off, slot, rank, projs, {s: 1.0 + s for s in range(len(ranks))})


@pytest.mark.parametrize("lens,slot,ranks", [
    ([77], [0], [32]),                                                        # one tile and a remainder of 13
    ([1, 64, 1, 16, 1], [1, 0, -1, 2, 1], [100, 5, 64]),                      # whole tiles, requests of pools too small for one, a row without adapter
    ([65, 1, 30, 8] + [1] * 40, [0, 1, 2, 3] + [4 + i % 5 for i in range(40)], [16, 33, 128, 8, 1, 17, 64, 96, 127]),  # pools of eight one-token requests become tiles too
    ([193, 7, 7, 7], [0, 1, 1, 2], [5, 65, 16]),                              # two segments of seven make a tile, one does not
])
def test_units(lens, slot, ranks):
    h, plan, batch = _plan(lens, slot, ranks, LAYER, 8)
    own = check_plan_units(h, plan, *batch)
    other = check_plan_units(h, plan, *batch, tiled=True)
    assert own[0]["tiles"] == 0 and other[0]["tiles"] > 0
    assert B.lora_plan_destroy(h, plan) == B.LORA_OK and B.lora_cache_destroy(h) == B.LORA_OK


@pytest.mark.parametrize("why,kw", [
    ("no tokens for a tile", dict(lens=[15] * 4, slot=[0, 1, 2, 3], ranks=[16] * 4, projs=LAYER, layers=8)),
    ("tiles of its own", dict(lens=[900, 800], slot=[0, 1], ranks=[128, 64], projs=LAYER, layers=8)),
    ("few tokens of a small projection: nothing gains", dict(lens=[16], slot=[0], ranks=[4], projs=[(64, 64)], layers=1)),
    ("a threshold of the caller's", dict(lens=[77], slot=[0], ranks=[32], projs=LAYER, layers=8, mfma_min_tokens=100)),
    ("fp32", dict(lens=[77], slot=[0], ranks=[32], projs=LAYER, layers=8, dtype=B.LORA_F32)),
    ("small scratch", dict(lens=[77], slot=[0], ranks=[32], projs=LAYER, layers=8, flags=B.LORA_CACHE_HOST_ONLY | B.LORA_CACHE_SMALL_SCRATCH)),
])
def test_plans_without(why, kw):
    h, plan, batch = _plan(**kw)
    if why != "small scratch":  # (such plans have no wide items)
        check_plan_units(h, plan, *batch, bf16=kw.get("dtype") != B.LORA_F32)
    rc, units, toks = B.lora_plan_dump_tiled(h, plan, 0)
    assert rc == B.LORA_OK and len(units) == 0 and len(toks) == 0
    assert B.lora_plan_destroy(h, plan) == B.LORA_OK
    assert B.lora_cache_destroy(h) == B.LORA_OK


def test_a_plan_made_in_anothers_place():
    h, plan, (T, off, slot, rank, projs, alpha) = _plan([77, 1, 1, 1], [0, 1, 1, 1], [32, 8], LAYER, 8, n_plans=1)
    check_plan_units(h, plan, T, off, slot, rank, projs, alpha, tiled=True)
    assert B.lora_plan_destroy(h, plan) == B.LORA_OK
    off2, slot2, rank2 = np.arange(5, dtype=np.int32), np.asarray([0, 1, -1, 1], np.int32), np.asarray([32, 8, 0, 8], np.int32)
    rc, plan = B.lora_plan_create(h, 4, off2, slot2, rank2)
    assert rc == B.LORA_OK
    check_plan_units(h, plan, 4, off2, slot2, rank2, projs, alpha)
    rc, units, _toks = B.lora_plan_dump_tiled(h, plan, 0)
    assert rc == B.LORA_OK and len(units) == 0
    assert B.lora_plan_destroy(h, plan) == B.LORA_OK and B.lora_cache_destroy(h) == B.LORA_OK
