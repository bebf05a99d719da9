"""lora_linear_plan where its grid can go wrong: tiles split along k into every number of parts (the sums of the parts of a
tile meet in its output), whole rounds before a split one, ragged panels, odd numbers of k stages."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _shape(B, pool, plan):
    """(rows of a tile, stages of a ring, tiles, tiles split along k, parts of each) of the plan's product of projection 0"""
    rc, units, _toks = B.lora_plan_dump(pool.handle, plan, 0)
    assert rc == B.LORA_OK
    (u,) = units[units["kind"] == B.LORA_UNIT_LINEAR_SHAPE]
    return int(u["lo"]), int(u["alpha"]), int(u["hi"]), int(u["where"]) >> 8, int(u["where"]) & 255


# (the shape on 256 compute units: on another part these cases test what they reach there)
@pytest.mark.parametrize("lens,h_in,h_out,shape", [
    ([300], 4096, 1024, (64, 4, 80, 80, 3)),                  # tiles of 64 x 64, split along k
    ([1000], 4160, 1280, (64, 4, 320, 0, 1)),                 # of 64 x 64, 65 k stages
    ([1, 100, 30], 512, 11072, (64, 3, 519, 0, 1)),           # of 64 x 64, more than fit side by side with a ring of four
    ([1, 700, 900, 2, 833], 2112, 1024, (128, 3, 320, 0, 1)), # of 128 x 64, 33 k stages, an odd number of runs
    ([740], 8256, 1024, (256, 2, 12, 12, 8)),                 # eight parts, 129 k stages
    ([700], 11008, 2304, (256, 2, 27, 27, 8)),                # eight parts, 172 k stages
    ([700], 6208, 1536, (256, 2, 18, 18, 7)),                 # seven parts, 97 k stages
    ([500], 8256, 3072, (256, 2, 36, 36, 6)),                 # six parts, 129 k stages
    ([1300], 4160, 1536, (256, 2, 36, 36, 5)),                # five parts, 65 k stages
    ([2300], 4160, 1088, (256, 2, 50, 50, 4)),                # four parts, the last column panel 64 wide
    ([1300], 2112, 2560, (256, 2, 60, 60, 3)),                # three parts, 33 k stages
    ([4000, 100], 4096, 1088, (256, 2, 85, 85, 3)),           # three parts, the last column panel 64 wide
    ([2306], 256, 4992, (256, 2, 200, 0, 1)),                 # whole, four k stages
    ([2000, 17], 4096, 4096, (256, 2, 128, 128, 2)),          # two parts
    ([1700], 4096, 4096, (256, 2, 112, 112, 2)),              # two parts
    ([3000, 462], 1600, 4928, (256, 2, 280, 24, 3)),          # a whole round, then 24 tiles in three parts, 25 k stages
    ([5084], 1536, 4736, (256, 2, 380, 124, 2)),              # a whole round, then 124 tiles in two parts
    ([8149], 1792, 2112, (256, 2, 288, 32, 4)),               # a whole round, then 32 tiles in four parts
    ([63], 64, 64, (64, 4, 2, 0, 1)),                         # one k stage
    ([65, 5], 192, 320, (64, 4, 10, 0, 1)),                   # three k stages
])
def test_linear_against_torch(lens, h_in, h_out, shape):
    check_against_torch(lens, h_in, h_out, shape)


# tiles of 192 and 288 rows: the last panel full, of one row more than a run of 64, one short; the last column panel 64 wide; odd k stages
@pytest.mark.parametrize("lens,h_in,h_out,shape", [
    ([2800, 35, 200, 17], 4096, 4096, (192, 2, 256, 0, 1)),    # 16 panels, all full
    ([1500, 1000, 9, 350], 2368, 4160, (192, 2, 255, 0, 1)),   # 37 k stages, ragged
    ([3500, 700, 71], 4096, 4096, (288, 2, 240, 0, 1)),        # the last panel 259 rows
    ([3500, 1025, 63], 2368, 4096, (288, 2, 256, 0, 1)),       # 16 panels, all full, 37 k stages
    ([2400, 140], 4096, 13376, (288, 2, 477, 0, 1)),           # two rounds, the last column panel 64 wide
    ([3100], 2048, 2432, (192, 2, 170, 0, 1)),                 # 32 k stages
    ([4096, 300], 2112, 4096, (288, 2, 256, 0, 1)),            # 33 k stages
    ([16384, 190], 512, 1024, (288, 2, 232, 0, 1)),            # eight k stages
    ([1271], 384, 7168, (192, 2, 196, 0, 1)),                  # six and seven k stages, as few as either size is taken for
    ([7182], 448, 1024, (192, 2, 152, 0, 1)),
    ([8942], 384, 2048, (288, 2, 256, 0, 1)),
    ([6961], 448, 2432, (288, 2, 250, 0, 1)),
])
@pytest.mark.parametrize("workspace", [True, False])
def test_tall_tiles_against_torch(lens, h_in, h_out, shape, workspace):
    check_against_torch(lens, h_in, h_out, shape, workspace)


def check_against_torch(lens, h_in, h_out, shape, workspace=True):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    ranks = [16, 128, 40]
    gen = torch.Generator(device="cuda").manual_seed(h_in + h_out + len(lens))
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    lens = lens + [1] * 20  # requests on the GEMV path, some without an adapter
    slot = np.asarray([i % 3 if i % 5 != 4 or lens[i] > 1 else -1 for i in range(len(lens))], np.int32)
    T = sum(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    A, Bm = [normal(h_in, r, sigma=0.02) for r in ranks], [normal(r, h_out, sigma=0.02) for r in ranks]
    x, wt = normal(T, h_in), normal(h_out, h_in, sigma=0.02)
    pool = LoraPool([(h_in, h_out)], 1, [128], [3], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=16)
    try:
        for i, r in enumerate(ranks):
            pool.fill(i, i + 1, r, 0.5 + i, 0, 0, A[i].cpu(), Bm[i].cpu())
        plan = pool.plan(T, off, slot, np.where(slot >= 0, np.asarray(ranks)[slot], 0).astype(np.int32))
        assert _shape(B, pool, plan) == shape or torch.cuda.get_device_properties(0).multi_processor_count != 256
        space = torch.empty(T * h_out, dtype=torch.float32, device="cuda")
        ref = x.double() @ wt.double().t()
        term = torch.zeros_like(ref)
        for g, s in enumerate(slot):
            if s >= 0:
                a, b = int(off[g]), int(off[g + 1])
                term[a:b] = 2.0 * (0.5 + s) * (x[a:b].double() @ A[s].double()) @ Bm[s].double()
        ref += term
        term[: -20] = 0  # (of the requests on the GEMV path)
        for _ in range(3):  # the counts of split tiles are back at zero after every launch
            y = torch.full((T, h_out), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.check(B.lora_linear_plan(pool.handle, plan, 0, 0, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0,
                                       torch.cuda.current_stream().cuda_stream, *((space.data_ptr(), space.numel() * 4) if workspace else ())))
            pool.check_fault()
            err, rms = (y.double() - ref).abs(), ref.pow(2).mean().sqrt()
            # one rounding of the output (half an ulp: 2^-9 of the element's binade, at most 2^-8 of its value) beside the
            # rounding of s.v to bf16 (2^-9 of each of its entries: well under 2^-8 of the RMS in the sum); without a workspace
            # the requests' adapter term is rounded by itself on its way (at most 2^-8 of it)
            assert bool((err <= 2.0**-8 * ref.abs() + 2.0**-7 * rms + (0 if workspace else 2.0**-8 * term.abs())).all()), float((err / rms).max())
            assert float((y.double() - ref).norm() / ref.norm()) < 4e-3
    finally:
        pool.close()


@pytest.mark.parametrize("h_in,h_out", [(64, 64), (192, 320), (1024, 1088), (1536, 1536), (4096, 256), (4096, 4096)])  # 4096 -> 256: split tiles of 64 x 64
@pytest.mark.parametrize("lens", [
    [8, 9, 15, 16, 17, 1, 1, 1, 31, 33],             # several slots in a run and in a block of 16 rows, GEMV and plain rows behind them
    [60, 8, 64, 8, 120, 1, 1],                       # segments that end one run and begin the next
    [250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1],    # across a panel of 256 rows
    [1] * 70 + [8],                                  # GEMV rows over two runs, the first beside a tile
    [700, 13, 8, 400, 1, 1, 1],                      # 1536 -> 1536: tiles of 128 x 64, an odd number of runs
])
def test_rows_of_several_slots(lens, h_in, h_out):
    check_rows_of_several_slots(lens, h_in, h_out)


@pytest.mark.parametrize("lens,h_in,h_out,rows", [
    ([250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1, 1748], 256, 4992, 256),
    ([250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1, 2500], 2048, 2432, 192),
    ([183, 12, 200, 1, 9, 17, 8, 40, 8, 8, 8, 8, 1, 8, 33] * 5 + [1] * 40, 2048, 2432, 192),
    ([250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1, 3818], 2112, 4096, 288),
    ([281, 12, 300, 1, 9, 17, 8, 40, 8, 8, 8, 8, 1, 8, 33] * 6 + [1] * 100, 2112, 4096, 288),
])
def test_rows_of_several_slots_in_tall_tiles(lens, h_in, h_out, rows):
    check_rows_of_several_slots(lens, h_in, h_out, rows)


def check_rows_of_several_slots(lens, h_in, h_out, rows=None):
    """Neighbouring segments differ in slot and rank (some no multiple of 8); the rows of the intermediate hold NaN behind their ranks."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    ranks = [5, 128, 33, 16, 100]
    gen = torch.Generator(device="cuda").manual_seed(h_in + len(lens))
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    T = sum(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ones = [i for i, n in enumerate(lens) if n == 1]
    slot = np.asarray([i % 5 if n > 1 else 5 + ones.index(i) % 30 for i, n in enumerate(lens)], np.int32)  # one-token requests: at most four of a slot
    slot[ones[1::7]] = -1
    rank_of = np.asarray(ranks + [ranks[i % 5] for i in range(30)])
    A, Bm = [normal(h_in, r, sigma=0.02) for r in rank_of], [normal(r, h_out, sigma=0.02) for r in rank_of]
    x, wt = normal(T, h_in), normal(h_out, h_in, sigma=0.02)
    pool = LoraPool([(h_in, h_out)], 1, [128], [35], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=8)
    try:
        pool.buf.fill_(0xFF)  # NaN in every word that is not written: the next pool takes the same memory, and what has to be zero there it clears
        pool.close()
        pool = LoraPool([(h_in, h_out)], 1, [128], [35], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=8)
        for i, r in enumerate(rank_of):
            pool.fill(i, i + 1, int(r), 0.5 + i % 3, 0, 0, A[i].cpu(), Bm[i].cpu())
        plan = pool.plan(T, off, slot, np.where(slot >= 0, rank_of[slot], 0).astype(np.int32))
        assert rows is None or _shape(B, pool, plan)[0] == rows or torch.cuda.get_device_properties(0).multi_processor_count != 256
        ref = x.double() @ wt.double().t()
        for g, s in enumerate(slot):
            if s >= 0:
                a, b = int(off[g]), int(off[g + 1])
                ref[a:b] += 2.0 * (0.5 + s % 3) * (x[a:b].double() @ A[s].double()) @ Bm[s].double()
        space = torch.full((T * h_out,), float("nan"), dtype=torch.float32, device="cuda")
        for _ in range(2):
            y = torch.full((T, h_out), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.check(B.lora_linear_plan(pool.handle, plan, 0, 0, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0,
                                       torch.cuda.current_stream().cuda_stream, space.data_ptr(), space.numel() * 4))
            pool.check_fault()
            err, rms = (y.double() - ref).abs(), ref.pow(2).mean().sqrt()
            assert bool((err <= 2.0**-8 * ref.abs() + 2.0**-7 * rms).all()), float((err / rms).max())  # as above
            assert float((y.double() - ref).norm() / ref.norm()) < 4e-3
    finally:
        pool.close()


@pytest.mark.parametrize("lens,h_in,h_out,shape", [
    ([8, 9, 15, 16, 17, 1, 1, 1, 31, 33], 1024, 1088, (64, 4, 1)),   # tiles of 64 x 64
    ([8, 9, 15, 16, 17, 1, 1, 1, 31, 33], 4096, 256, (64, 4, 5)),    # of 64 x 64, split along k
    ([8, 9, 15, 16, 17, 1, 1, 1, 31, 33], 512, 11072, (64, 3, 1)),   # of 64 x 64, more of them than fit side by side with a ring of four
    ([700, 13, 8, 400, 1, 1, 1], 1536, 1536, (128, 3, 1)),           # of 128 x 64
    ([700, 13, 8, 400, 1, 1, 1], 4096, 4096, (256, 2, 3)),           # of 256 x 256, split along k
    ([250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1, 1748], 256, 4992, (256, 2, 1)),   # of 256 x 256, whole
    ([250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1, 2500], 2048, 2432, (192, 2, 1)),  # of 192 x 256
    ([250, 12, 250, 1, 8, 8, 8, 8, 8, 8, 8, 8, 1, 3818], 2112, 4096, (288, 2, 1)),  # of 288 x 256
])
def test_infinities_stay_with_their_adapter(lens, h_in, h_out, shape):
    """Infinities and NaN in one adapter's B: the rows of every other segment, of the requests on the GEMV path and of those without
    an adapter are bit for bit what they are beside the same adapter with finite weights, whichever block of 16 rows they share
    with it; so are its own rows in the columns that are finite."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    ranks = [5, 128, 33, 16, 100]
    gen = torch.Generator(device="cuda").manual_seed(h_in + len(lens))
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    T = sum(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ones = [i for i, n in enumerate(lens) if n == 1]
    slot = np.asarray([i % 5 if n > 1 else 5 + ones.index(i) for i, n in enumerate(lens)], np.int32)
    slot[ones[1:2]] = -1
    rank_of = np.asarray(ranks + [ranks[i % 5] for i in range(len(ones))])
    A, Bm = [normal(h_in, r, sigma=0.02) for r in rank_of], [normal(r, h_out, sigma=0.02) for r in rank_of]
    x, wt = normal(T, h_in), normal(h_out, h_in, sigma=0.02)
    space = torch.empty(T * h_out, dtype=torch.float32, device="cuda")
    slot_of_token = torch.as_tensor(np.repeat(slot, lens), device="cuda")
    pool = LoraPool([(h_in, h_out)], 1, [128], [len(rank_of)], B.LORA_BF16, max_tokens=T, max_segments=len(lens), mfma_min_tokens=8)
    try:
        def product(bad):
            for i, r in enumerate(rank_of):
                w = Bm[i].clone()
                if i == bad:
                    w[0, 0::4], w[-1, 1::4], w[r // 2, 2::4] = float("inf"), float("nan"), float("-inf")
                B.lora_cache_release_slot(pool.handle, i)
                pool.fill(i, i + 1, int(r), 1.0, 0, 0, A[i].cpu(), w.cpu())
            torch.cuda.synchronize()
            plan = pool.plan(T, off, slot, np.where(slot >= 0, rank_of[slot], 0).astype(np.int32))
            rows, ring, _tiles, _split, parts = _shape(B, pool, plan)
            assert (rows, ring, parts) == shape or torch.cuda.get_device_properties(0).multi_processor_count != 256
            y = torch.full((T, h_out), 7.0, dtype=torch.bfloat16, device="cuda")
            B.check(B.lora_linear_plan(pool.handle, plan, 0, 0, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0,
                                       torch.cuda.current_stream().cuda_stream, space.data_ptr(), space.numel() * 4))
            pool.check_fault()
            pool.plan_destroy(plan)
            return y

        want = product(-1)
        assert bool(want.isfinite().all())
        for bad in sorted({int(s) for s in slot if 0 <= s < 5}):
            got, own = product(bad), slot_of_token == bad
            assert torch.equal(got[~own], want[~own]), f"{int((got[~own] != want[~own]).sum())} values beside slot {bad}"
            assert torch.equal(got[own][:, 3::4], want[own][:, 3::4])
            assert not bool(got[own][:, 1::4].isfinite().any())
    finally:
        pool.close()


@pytest.mark.parametrize("T,h_in,h_out,tiles", [(760, 8256, 1024, 12), (700, 11008, 2304, 27), (1100, 4096, 4096, 80), (2048, 4096, 4096, 128)])
def test_tiles_finished_by_the_last_part_alone(T, h_in, h_out, tiles):
    """What happens when a part is done before another has started, forced from the host: the tiles' state (16 bytes each,
    behind the slabs: parts started, way, parts arrived, parts that have read) says so before the launch.  Bit for bit the
    result of parts that share the tile; the state is back at zero."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    pool = LoraPool([(h_in, h_out)], 1, [16], [1], B.LORA_BF16, max_tokens=T, max_segments=1)
    try:
        pool.fill(0, 1, 16, 1.0, 0, 0, normal(h_in, 16, sigma=0.02).cpu(), normal(16, h_out, sigma=0.02).cpu())
        plan = pool.plan(T, np.asarray([0, T], np.int32), np.zeros(1, np.int32), np.full(1, 16, np.int32))
        assert _shape(B, pool, plan)[::2] == (256, tiles, _shape(B, pool, plan)[4]) and _shape(B, pool, plan)[3] == tiles
        x, wt = normal(T, h_in), normal(h_out, h_in, sigma=0.02)
        _rc, slab, n = B.lora_cache_slab(pool.handle, 0, 0, 0)
        state = pool.buf[slab + n - pool.buf.data_ptr():][: 16 * tiles].view(torch.int32).view(tiles, 4)
        assert (slab + n) % 256 == 0
        outs = []
        for way in (0, 2, 0, 2):
            y = torch.full((T, h_out), float("nan"), dtype=torch.bfloat16, device="cuda")
            assert not state.any()
            state[:, 1] = way
            B.check(B.lora_linear_plan(pool.handle, plan, 0, 0, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0, torch.cuda.current_stream().cuda_stream))
            pool.check_fault()
            outs.append(y)
        assert not state.any()
        assert not outs[0].isnan().any()
        for y in outs[1:]:
            assert torch.equal(y, outs[0])
    finally:
        pool.close()


@pytest.mark.parametrize("T,h,h_out,shape", [(1100, 4096, 4096, (256, 2, 80, 80, 3)), (300, 4096, 1024, (64, 4, 80, 80, 3))])
def test_split_products_on_a_busy_device(T, h, h_out, shape):
    """Launches whose last round is all parts of split tiles (80 tiles of three parts) from two caches on two streams beside
    matrix products on a third: parts get their places late and in whatever order, and a tile whose parts are not all running
    when its first part is done is finished by the last of them alone (tiles of 64 x 64 always are: there the last part may
    find the others' sums before it has left its own, or after).  The results are those of one launch by itself, bit for bit."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    rank, n = 16, 24
    gen = torch.Generator(device="cuda").manual_seed(7)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    A, Bm = normal(h, rank, sigma=0.02).cpu(), normal(rank, h_out, sigma=0.02).cpu()
    x, wt = [normal(T, h) for _ in range(2)], [normal(h_out, h, sigma=0.02) for _ in range(2)]
    y = [[torch.empty(T, h_out, dtype=torch.bfloat16, device="cuda") for _ in range(n)] for _ in range(2)]
    a, b, c = normal(2048, 2048), normal(2048, 2048), torch.empty(2048, 2048, dtype=torch.bfloat16, device="cuda")
    pools = [LoraPool([(h, h_out)], 1, [rank], [1], B.LORA_BF16, max_tokens=T, max_segments=1) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(3)]
    try:
        plans = []
        for q in pools:
            q.fill(0, 1, rank, 1.0, 0, 0, A, Bm)
            plans.append(q.plan(T, np.asarray([0, T], np.int32), np.zeros(1, np.int32), np.full(1, rank, np.int32)))
        assert _shape(B, pools[0], plans[0]) == shape or torch.cuda.get_device_properties(0).multi_processor_count != 256
        torch.mm(a, b, out=c)
        torch.cuda.synchronize()

        def product(k, i):
            B.check(B.lora_linear_plan(pools[k].handle, plans[k], 0, 0, x[k].data_ptr(), wt[k].data_ptr(), y[k][i].data_ptr(), 2.0, streams[k].cuda_stream))

        want = []
        for k in range(2):
            product(k, 0)
            torch.cuda.synchronize()
            want.append(y[k][0].clone())
            y[k][0].zero_()
        torch.cuda.synchronize()
        for i in range(n):
            with torch.cuda.stream(streams[2]):
                for _ in range(4):
                    torch.mm(a, b, out=c)
            for k in range(2):
                product(k, i)
        torch.cuda.synchronize()
        for k in range(2):
            pools[k].check_fault(streams[k])
            for i in range(n):
                assert torch.equal(y[k][i], want[k]), (k, i)
    finally:
        for q in pools:
            q.close()
