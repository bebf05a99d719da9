"""lora_apply_plan_multi as batches (one launch per phase for all entries that do not depend on each other) against one
lora_apply_plan per entry, where batches can go wrong: more entries than a batch holds, groups of every size, rows and columns
of different lengths, few and many GEMV items, few and many tiles, entries that depend on earlier ones, capture."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

PROJS = [(512, 512), (512, 512), (512, 192), (512, 1088), (512, 512), (512, 64), (192, 512), (1088, 512), (2112, 2240)]  # 0..5 read one x
# lengths, ranks, tokens from which tiles are formed, tokens per slot (None: dealt out in turn, every seventh without an adapter)
BATCHES = {
    "one token": ([1], [16], 8, None),
    "decode": ([1] * 90, [8, 16, 12, 32, 64, 96, 128, 33], 8, None),
    "decode, no tiles": ([1] * 90, [8, 16, 12, 32, 64, 96, 128, 33], 1000, None),  # more than 64 shrink items
    # every number of tokens of an item and its remainders, with ranks of every body: 8 and 16 rows, 1 to 4 k steps
    "popular": (None, [8, 16, 24, 32, 5, 12, 100, 128, 64, 33, 40, 72], 1000, [1, 2, 3, 4, 5, 8, 9, 12, 16, 17, 7, 35]),
    "popular, other ranks": (None, [128, 100, 64, 33, 8, 3, 16, 11, 24, 8, 16, 8], 1000, [1, 2, 3, 4, 5, 8, 9, 12, 16, 17, 7, 35]),
    "few prompts": ([77, 9], [16, 128], 8, None),
    "tiles of a few tokens": ([9, 10, 11, 12, 13, 14, 15, 8] * 3, [8, 40, 128], 8, None),
    "mixed": ([300, 1, 65, 1, 1, 17, 128, 1, 3, 1, 200], [16, 64, 128, 8], 8, None),
}


def _setup(lens, ranks, m0, counts, layers, dtype="bf16", flags=0):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    if counts:
        slot = np.random.default_rng(1).permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)
        lens = [1] * len(slot)
    else:
        slot = np.asarray([i % len(ranks) if i % 7 != 6 else -1 for i in range(len(lens))], np.int32)
    T = sum(lens)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(len(lens) + layers)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda", dtype=dt).mul_(sigma)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    pool = LoraPool(PROJS, layers, [128], [len(ranks)], B.LORA_BF16 if dtype == "bf16" else B.LORA_F32, max_tokens=T,
                    max_segments=len(lens), mfma_min_tokens=m0 if dtype == "bf16" else 0, flags=flags)
    for s, r in enumerate(ranks):
        for layer in range(layers):
            for p, (h_in, h_out) in enumerate(PROJS):
                pool.fill(s, s + 1, r, 0.5 + s, layer, p, normal(h_in, r, sigma=0.05).cpu(), normal(r, h_out, sigma=0.05).cpu())
    torch.cuda.synchronize()
    plan = pool.plan(T, off, slot, np.where(slot >= 0, np.asarray(ranks)[slot], 0).astype(np.int32))
    return B, pool, plan, T, normal


def _same(got, want, dtype, what):
    """The sums may be split in other places: the intermediate then rounds elsewhere once in a while (2^-9 of an entry, well
    under 2^-8 of the RMS in the sum) and the output by up to two halves of its last place."""
    got, want = got.double(), want.double()
    rms = want.pow(2).mean().sqrt()
    rel, floor = (2.0**-7, 2.0**-7) if dtype == "bf16" else (2.0**-21, 2.0**-20)
    err = (got - want).abs()
    assert bool((err <= rel * want.abs() + floor * rms).all()), f"{what}: {float((err / rms).max())}"


@pytest.mark.parametrize("dtype,flags", [("bf16", "auto"), ("bf16", "split"), ("f32", "auto")])
@pytest.mark.parametrize("batch", list(BATCHES))
def test_batches_against_single_applies(batch, dtype, flags):
    from paper_2411_17741_amd import binding as B0

    layers = 14
    assert layers * len(PROJS) > 120  # more than a batch holds, of GEMV work alone or with tiles
    fl = B0.LORA_CACHE_SPLIT_GEMV if flags == "split" else 0
    B, pool, plan, T, normal = _setup(*BATCHES[batch], layers, dtype, fl)
    try:
        xs = [normal(T, 512), normal(T, 192), normal(T, 1088), normal(T, 2112)]
        x_of = lambda p: xs[0 if p < 6 else p - 5]
        sh = torch.cuda.current_stream().cuda_stream
        base = [[normal(T, h_out) for _i, h_out in PROJS] for _ in range(layers)]
        want = [[y.clone() for y in ys] for ys in base]
        for layer in range(layers):
            for p in range(len(PROJS)):
                pool.apply_plan(plan, layer, p, x_of(p), want[layer][p], 2.0)
        for _ in range(2):  # again with the scratch as the first call left it
            got = [[y.clone() for y in ys] for ys in base]
            descs = B.make_descs([(l, p, x_of(p).data_ptr(), got[l][p].data_ptr()) for l in range(layers) for p in range(len(PROJS))])
            B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, sh))
            pool.check_fault()
            for l in range(layers):
                for p in range(len(PROJS)):
                    assert not torch.equal(got[l][p], base[l][p])
                    _same(got[l][p], want[l][p], dtype, f"layer {l} projection {p}")
    finally:
        pool.close()


@pytest.mark.parametrize("batch", ["popular", "mixed"])
@pytest.mark.parametrize("how", ["flag", "fewer bytes"])
def test_small_scratch(batch, how, monkeypatch):
    """A pool with the scratch of four projections, asked for or found too small for more: lists, single applies and the
    fused product give what they give in a full pool; a byte less is refused."""
    from paper_2411_17741_amd import binding as B0

    required = B0.lora_cache_bytes_required
    outs, sizes = [], []
    for small in (False, True):
        flags = 0
        if small and how == "flag":
            flags = B0.LORA_CACHE_SMALL_SCRATCH
        elif small:
            def fewer(cfg):
                cfg.flags |= B0.LORA_CACHE_SMALL_SCRATCH
                n = required(cfg)
                cfg.flags &= ~B0.LORA_CACHE_SMALL_SCRATCH
                return n
            monkeypatch.setattr(B0, "lora_cache_bytes_required", fewer)
        B, pool, plan, T, normal = _setup(*BATCHES[batch], 3, flags=flags)
        sizes.append(pool.bytes)
        try:
            xs = [normal(T, 512), normal(T, 192), normal(T, 1088), normal(T, 2112)]
            x_of = lambda p: xs[0 if p < 6 else p - 5]
            sh = torch.cuda.current_stream().cuda_stream
            y = [[normal(T, h_out) for _i, h_out in PROJS] for _ in range(3)]
            descs = B.make_descs([(l, p, x_of(p).data_ptr(), y[l][p].data_ptr()) for l in range(3) for p in range(len(PROJS))])
            B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, sh))
            wt, z = normal(2240, 2112, sigma=0.05), torch.empty(T, 2240, dtype=torch.bfloat16, device="cuda")
            B.check(B.lora_linear_plan(pool.handle, plan, 0, 8, xs[3].data_ptr(), wt.data_ptr(), z.data_ptr(), 2.0, sh))
            pool.apply_plan(plan, 0, 8, xs[3], y[0][8], 2.0)
            pool.check_fault()
            outs.append([t for ys in y for t in ys] + [z])
            if small:
                rc, _h = B.lora_cache_create(pool.cfg, (pool.buf.data_ptr() + 255) // 256 * 256, pool.bytes - 1)
                assert rc == B.LORA_E_NOMEM
        finally:
            pool.close()
    assert sizes[1] < sizes[0]
    for k, (got, want) in enumerate(zip(outs[1], outs[0])):
        _same(got, want, "bf16", f"output {k}")


@pytest.mark.parametrize("batch", ["popular", "mixed"])
def test_a_pool_with_room_for_fewer_sets(batch, monkeypatch):
    """A pool of fewer bytes than are required runs lists as batches of as many projections as it has room for, not four at a time:
    a byte short, and 14 sets short.  The results are those of a full pool."""
    from paper_2411_17741_amd import binding as B0

    required = B0.lora_cache_bytes_required

    def smallest(cfg):
        cfg.flags |= B0.LORA_CACHE_SMALL_SCRATCH
        n = required(cfg)
        cfg.flags &= ~B0.LORA_CACHE_SMALL_SCRATCH
        return n

    sizes = [required, lambda cfg: required(cfg) - 1, lambda cfg: required(cfg) - 14 * 1024 * cfg.max_tokens, smallest]  # (a set has 1 KB per token)
    entries, outs = [], []
    for size in sizes:
        monkeypatch.setattr(B0, "lora_cache_bytes_required", size)
        B, pool, plan, T, normal = _setup(*BATCHES[batch], 2)
        try:
            xs = [normal(T, 512), normal(T, 192), normal(T, 1088), normal(T, 2112)]
            y = [normal(T, h_out) for _ in range(2) for _i, h_out in PROJS]
            descs = B.make_descs([(l, p, xs[0 if p < 6 else p - 5].data_ptr(), y[l * len(PROJS) + p].data_ptr()) for l in range(2) for p in range(len(PROJS))])
            B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
            pool.check_fault()
            n = 0
            for p in range(len(PROJS)):  # entries of the first batch
                rc, units, _toks = B.lora_plan_dump(pool.handle, plan, p)
                assert rc == B.LORA_OK
                n += len(set(int(w) for w in units[units["kind"] == B.LORA_UNIT_BATCH_SHRINK]["where"]))
            entries.append(n)
            outs.append(y)
        finally:
            pool.close()
    assert entries[0] == 18 and entries[1] == 18 and 4 < entries[2] < 18 and entries[3] == 4, entries
    for y in outs[1:]:
        for k, (got, want) in enumerate(zip(y, outs[0])):
            _same(got, want, "bf16", f"output {k}")


@pytest.mark.parametrize("batch", ["decode", "decode, no tiles", "mixed"])
def test_entries_that_depend_on_earlier_ones(batch):
    """Each list in order: an output that is a later entry's input; a later output over an earlier input; one output twice;
    an output that overlaps another's last row; an entry in place."""
    B, pool, plan, T, normal = _setup(*BATCHES[batch], 2)
    try:
        sh = torch.cuda.current_stream().cuda_stream

        def fresh(seed):
            g = torch.Generator(device="cuda").manual_seed(seed)
            return [torch.randn(2 * T, 512, generator=g, device="cuda").bfloat16() for _ in range(4)]

        at = lambda t, row=0: t.data_ptr() + row * t.shape[1] * 2
        lists = [
            lambda t: [(0, 0, at(t[0]), at(t[1])), (1, 0, at(t[1]), at(t[2])), (1, 1, at(t[2]), at(t[3]))],
            lambda t: [(0, 0, at(t[0]), at(t[1])), (1, 0, at(t[2]), at(t[0])), (1, 1, at(t[0]), at(t[3]))],
            lambda t: [(0, 0, at(t[0]), at(t[1])), (0, 1, at(t[0]), at(t[1])), (1, 4, at(t[2]), at(t[1]))],
            lambda t: [(0, 0, at(t[0]), at(t[1])), (1, 0, at(t[0]), at(t[1], T - 1)), (1, 1, at(t[1], T - 1), at(t[2]))],
            lambda t: [(0, 1, at(t[3]), at(t[2])), (0, 0, at(t[0]), at(t[0])), (1, 0, at(t[0]), at(t[1]))],
        ]
        # (in place with as many columns out as in: a token's row is written when all of its words are there, that is when
        # everything that reads the row has read it)
        for n, make in enumerate(lists):
            want, got = fresh(n), fresh(n)
            for layer, p, x, y in make(want):
                B.check(B.lora_apply_plan(pool.handle, plan, layer, p, x, y, 2.0, sh))
            B.check(B.lora_apply_plan_multi(pool.handle, plan, B.make_descs(make(got)), 2.0, sh))
            pool.check_fault()
            for k, (a, b) in enumerate(zip(got, want)):
                _same(a, b, "bf16", f"list {n}, tensor {k}")
    finally:
        pool.close()


def _replays_match(pool, xs, prepare, call, outputs):
    """Captures call() and replays it with other activations each time, nothing enqueued on the cache in between: a replay that
    took the hand-over words of the replay before for its own would give that one's results.  Every replay against the eager
    call on the same activations, made before the capture."""
    from paper_2411_17741_amd import binding as B

    versions = [[x * f for x in xs] for f in (1.0, -0.5, 2.0, 1.0, 0.25)]
    want = []
    for v in versions:
        for x, value in zip(xs, v):
            x.copy_(value)
        prepare()
        call()
        pool.check_fault()
        want.append([t.clone() for t in outputs])
    assert not torch.equal(want[0][0], want[1][0])
    B.check(B.lora_cache_set_fencing(pool.handle, 0))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        call()
    B.check(B.lora_cache_set_fencing(pool.handle, 1))
    for v, w in zip(versions, want):
        for x, value in zip(xs, v):  # eager work between the replays
            x.copy_(value)
        prepare()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        pool.check_fault()
        for k, (a, b) in enumerate(zip(outputs, w)):
            assert torch.equal(a, b), f"output {k}"


# items and wide items, several token counts and ranks, tiles beside them; 126 entries: two batches at least, the second with fewer projections than
# the first (120 of GEMV work alone, then 6)
@pytest.mark.parametrize("batch,layers", [("one token", 3), ("decode", 3), ("popular", 3), ("mixed", 3), ("one token", 14), ("decode, no tiles", 14),
                                          ("popular", 14), ("decode", 14)])
def test_a_captured_batch_replays(batch, layers):
    B, pool, plan, T, normal = _setup(*BATCHES[batch], layers)
    try:
        xs = [normal(T, 512), normal(T, 192), normal(T, 1088), normal(T, 2112)]
        x_of = lambda p: xs[0 if p < 6 else p - 5]
        assert layers == 3 or layers * len(PROJS) > 120
        base = [normal(T, h_out) for _ in range(layers) for _i, h_out in PROJS]
        y = [t.clone() for t in base]
        descs = B.make_descs([(l, p, x_of(p).data_ptr(), y[l * len(PROJS) + p].data_ptr()) for l in range(layers) for p in range(len(PROJS))])
        _replays_match(pool, xs, lambda: [t.copy_(b) for t, b in zip(y, base)],
                       lambda: B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream)), y)
    finally:
        pool.close()


@pytest.mark.parametrize("workspace", [True, False])
@pytest.mark.parametrize("batch", ["one token", "mixed", "requests"])
def test_a_captured_linear_replays(batch, workspace):
    """The fused product's GEMV launch under capture: items, beside tiles, and wide items."""
    if batch == "requests":
        ranks, counts = _many_requests()
        assert _wide_items(counts, ranks) >= 600  # wide from 512
        B, pool, plan, T, normal = _setup(None, ranks, 1000, counts, 1)
    else:
        B, pool, plan, T, normal = _setup(*BATCHES[batch], 1)
    try:
        p = 3
        h_in, h_out = PROJS[p]
        x, wt, y = normal(T, h_in), normal(h_out, h_in, sigma=0.05), torch.empty(T, h_out, dtype=torch.bfloat16, device="cuda")
        space = torch.empty(T * h_out, dtype=torch.float32, device="cuda")
        _replays_match(pool, [x], lambda: y.fill_(float("nan")),
                       lambda: B.check(B.lora_linear_plan(pool.handle, plan, 0, p, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0,
                                                          torch.cuda.current_stream().cuda_stream, space.data_ptr() if workspace else 0,
                                                          space.numel() * 4 if workspace else 0)), [y])
    finally:
        pool.close()


def _many_requests():
    ranks = [8, 16, 24, 32, 5, 12, 100, 128, 64, 33, 40, 72] * 12
    return ranks, [1 + (5 * i) % 19 for i in range(len(ranks))]


def _wide_items(counts, ranks):
    """Wide shrink items (8 tokens, 16 stored rank rows) of so many one-token requests per slot."""
    return sum(-(-n // 8) * -(-(-(-r // 8) * 8) // 16) for n, r in zip(counts, ranks))


@pytest.mark.parametrize("workspace", [True, False])
@pytest.mark.parametrize("n_prompt", [0, 130])
def test_linear_with_many_requests(n_prompt, workspace):
    """The adapter term of requests in numbers that take wide items, as fp32 into the workspace or into the zeroed rows,
    beside the tile shrink of a prompt or without one."""
    ranks, counts = _many_requests()
    B, pool, plan, T, normal = _setup(None, ranks, 100 if n_prompt else 1000, counts, 1)
    pool.plan_destroy(plan)
    try:
        slot = np.random.default_rng(1).permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)
        lens = np.ones(len(slot), np.int32)
        if n_prompt:
            lens[7] = n_prompt  # one of the requests as a prompt, the last ones left out
            lens = lens[: len(slot) - n_prompt + 1]
            slot = slot[: len(lens)]
        requests = np.bincount(slot, minlength=len(ranks))
        if n_prompt:
            requests[slot[7]] = 0  # (in tiles)
        assert _wide_items(requests, ranks) >= 600  # wide from 512
        off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        plan = pool.plan(int(off[-1]), off, slot, np.asarray(ranks, np.int32)[slot])
        T, p = int(off[-1]), 3
        h_in, h_out = PROJS[p]
        x, wt, zeros = normal(T, h_in), normal(h_out, h_in, sigma=0.05), torch.zeros(T, h_out, dtype=torch.bfloat16, device="cuda")
        sh = torch.cuda.current_stream().cuda_stream
        space = torch.empty(T * h_out, dtype=torch.float32, device="cuda")
        pool.apply_plan(plan, 0, p, x, zeros, 2.0)  # the adapter terms alone, each rounded once
        want = x.double() @ wt.double().t() + zeros.double()
        for _ in range(2):
            y = torch.full((T, h_out), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.check(B.lora_linear_plan(pool.handle, plan, 0, p, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0, sh,
                                       space.data_ptr() if workspace else 0, space.numel() * 4 if workspace else 0))
            pool.check_fault()
            _same(y, want, "bf16", f"prompt {n_prompt}, workspace {workspace}")
    finally:
        pool.close()


@pytest.mark.parametrize("split", [False, True])
def test_a_list_large_enough_for_the_side_stream(split):
    """From 4 GB of the tile tokens' activations and outputs in a batch up the GEMV launch runs beside the tile kernels: eager and replayed,
    with the GEMV phases as one launch and as two, bit for bit what the same kernels give on one stream."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    h, layers, ranks = 4096, 32, [16, 128, 40, 8]
    lens = [1800, 1800, 1801] + [1] * 90
    slot = np.asarray([i % 4 if i % 7 != 6 else -1 for i in range(len(lens))], np.int32)
    T = sum(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(5)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(sigma)
    A, Bm = [normal(h, r, sigma=0.02).cpu() for r in ranks], [normal(r, h, sigma=0.02).cpu() for r in ranks]
    x = normal(T, h)
    base = normal(layers, T, h)
    y = base.clone()
    outs = []
    for flags in (B.LORA_CACHE_NO_OVERLAP, 0):
        flags |= B.LORA_CACHE_SPLIT_GEMV if split else 0
        pool = LoraPool([(h, h)], layers, [128], [4], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=100, flags=flags)
        try:
            for layer in range(layers):
                for s, r in enumerate(ranks):
                    pool.fill(s, s + 1, r, 0.5 + s, layer, 0, A[s], Bm[s])
            torch.cuda.synchronize()
            plan = pool.plan(T, off, slot, np.where(slot >= 0, np.asarray(ranks)[slot], 0).astype(np.int32))
            rc, units, _toks = B.lora_plan_dump(pool.handle, plan, 0)
            assert rc == B.LORA_OK and (units["kind"] == B.LORA_UNIT_GEMV_SHRINK).any()
            n_tile = int(units[units["kind"] == B.LORA_UNIT_TILE]["n_tok"].sum())
            runs = units[(units["kind"] == B.LORA_UNIT_TILE_SHRINK) & (units["where"] >> 20 == 6)]["where"] & 0xFFFFF
            assert layers * 2 * n_tile * 3 * h >= 4e9 and runs.max() < 32  # the 32 projections are one batch: 1024 runs
            descs = B.make_descs([(layer, 0, x.data_ptr(), y[layer].data_ptr()) for layer in range(layers)])
            call = lambda: B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
            y.copy_(base)
            call()
            torch.cuda.synchronize()
            pool.check_fault()
            outs.append(y.clone())
            if not flags & B.LORA_CACHE_NO_OVERLAP:
                _replays_match(pool, [x], lambda: y.copy_(base), call, [y])
        finally:
            pool.close()
    assert torch.equal(outs[0], outs[1]) and not torch.equal(outs[0], base)
