"""The tile shrink of short launches (units of 16 tokens x 16 rank rows, whole input rows) at the edges of its units, stages and wavefront shares,
one projection at a time and as lists, with the run table's kernel (small scratch) beside it."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_layers", [1, 5])  # 5: a batch's kernels
@pytest.mark.parametrize("h_in,h_out", [(64, 64), (192, 320), (448, 128), (1088, 1024), (4096, 512)])  # 1, 3, 7, 17 and 64 stages of 64 k
@pytest.mark.parametrize("lens", [[8], [16, 17, 9], [63, 64, 65, 1, 1], [300, 40, 128, 15, 1, 8]])
def test_short_tile_launches(lens, h_in, h_out, n_layers):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    ranks = [16, 5, 128, 33, 100, 8]
    gen = torch.Generator(device="cuda").manual_seed(h_in + len(lens))
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    T, n = sum(lens), len(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    A = [[normal(h_in, r, sigma=0.02) for r in ranks[:n]] for _ in range(n_layers)]
    Bm = [[normal(r, h_out, sigma=0.02) for r in ranks[:n]] for _ in range(n_layers)]
    x, base = [normal(T, h_in) for _ in range(n_layers)], [normal(T, h_out) for _ in range(n_layers)]
    for flags in (0, B.LORA_CACHE_SMALL_SCRATCH):
        make = lambda: LoraPool([(h_in, h_out)], n_layers, [128], [n], B.LORA_BF16, max_tokens=T, max_segments=n, mfma_min_tokens=8, flags=flags)
        pool = make()
        pool.buf.fill_(0xFF)  # NaN in every word that is not written: the next pool takes the same memory
        pool.close()
        pool = make()
        try:
            for layer in range(n_layers):
                for i in range(n):
                    pool.fill(i, i + 1, ranks[i], 0.5 + i, layer, 0, A[layer][i].cpu(), Bm[layer][i].cpu())
            plan = pool.plan(T, off, np.arange(n, dtype=np.int32), np.asarray(ranks[:n], np.int32))
            y = [b.clone() for b in base]
            descs = B.make_descs([(layer, 0, x[layer].data_ptr(), y[layer].data_ptr()) for layer in range(n_layers)])
            B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
            pool.check_fault()
            for layer in range(n_layers):
                ref, rounding = base[layer].double(), torch.zeros(T, h_out, dtype=torch.float64, device="cuda")
                for i in range(n):
                    a, b = int(off[i]), int(off[i + 1])
                    v = 2.0 * (0.5 + i) * (x[layer][a:b].double() @ A[layer][i].double())
                    ref[a:b] += v @ Bm[layer][i].double()
                    rounding[a:b] = v.abs() @ Bm[layer][i].double().abs()
                # the rounding of the output (2^-8 of its value) and that of every entry of s.v (2^-8 of its term); an eighth more for the sums in fp32
                assert bool(((y[layer].double() - ref).abs() <= 1.125 * 2.0**-8 * (ref.abs() + rounding)).all())
                assert float((y[layer].double() - ref).norm() / ref.norm()) < 4e-3
        finally:
            pool.close()


@pytest.mark.parametrize("h_in", [64, 192, 448])  # 1, 3 and 7 stages of 64 k
@pytest.mark.parametrize("ranks", [(8, 33, 80), (24, 64, 128), (16, 96, 5)])  # one to eight blocks of 16 rank rows
def test_whole_tiles_of_a_slot_in_pairs(h_in, ranks):
    """A list of 40 projections over 133 tiles, whole tiles of a slot behind each other: prompts with an odd number of tiles and ragged ends, and a pool of
    one-token requests of one slot."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    n_layers, h_out = 40, 64
    lens = [3000, 1, 2000, 650] + [1] * 300 + [2200, 500]
    slot = np.asarray([0, 2, 1, 2] + [2] * 300 + [1, 0], np.int32)
    gen = torch.Generator(device="cuda").manual_seed(h_in + ranks[0])
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    T, n = sum(lens), len(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    which = torch.from_numpy(np.repeat(slot, lens)).cuda()
    A, Bm = [normal(h_in, r, sigma=0.1) for r in ranks], [normal(r, h_out, sigma=0.1) for r in ranks]
    x, base = normal(T, h_in), normal(T, h_out)
    pool = LoraPool([(h_in, h_out)], n_layers, [128], [3], B.LORA_BF16, max_tokens=T, max_segments=n, mfma_min_tokens=8)
    try:
        for layer in range(n_layers):
            for i, r in enumerate(ranks):
                pool.fill(i, i + 1, r, 0.5 + i, layer, 0, A[i].cpu(), Bm[i].cpu())
        plan = pool.plan(T, off, slot, np.asarray(ranks, np.int32)[slot])
        _rc, units, _toks = B.lora_plan_dump(pool.handle, plan, 0)
        whole = [(u["where"], u["slot"]) for u in units if u["kind"] == B.LORA_UNIT_TILE_SHRINK and u["where"] >> 20 == 6 and u["alpha"] == -1]
        assert sum(a == b for a, b in zip(whole, whole[1:])) > 20
        y = [base.clone() for _ in range(n_layers)]
        descs = B.make_descs([(layer, 0, x.data_ptr(), y[layer].data_ptr()) for layer in range(n_layers)])
        B.check(B.lora_apply_plan_multi(pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
        pool.check_fault()
        ref, rounding = base.double(), torch.zeros(T, h_out, dtype=torch.float64, device="cuda")
        for i in range(3):
            v = 2.0 * (0.5 + i) * (x[which == i].double() @ A[i].double())
            ref[which == i] += v @ Bm[i].double()
            rounding[which == i] = v.abs() @ Bm[i].double().abs()
        for layer in range(n_layers):
            assert bool(((y[layer].double() - ref).abs() <= 1.125 * 2.0**-8 * (ref.abs() + rounding)).all()), layer  # as above
    finally:
        pool.close()
