"""lora_linear_plan where its grid can go wrong: tiles split along k into every number of parts (the sums of the parts of a
tile meet in its output), whole rounds before a split one, ragged panels, odd numbers of k stages."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,h_in,h_out", [
    ([300], 4096, 1024),                     # 8 tiles of 256 x 256: three parts
    ([300], 8192, 1024),                     # 8 tiles, 128 k stages: four parts
    ([1000], 4160, 1280),                    # 25 tiles, 65 k stages: three parts
    ([1, 700, 900, 2, 833], 2112, 1024),     # 44 tiles, 33 k stages: two parts
    ([4000, 100], 4096, 1088),               # 85 tiles, the last column panel 64 wide: two parts
    ([3100], 2048, 2432),                    # 130 tiles: whole
    ([2000, 17], 4096, 4096),                # 144 tiles: whole
    ([4096, 300], 2112, 4096),               # a whole round, then 32 tiles in two parts
    ([16384, 190], 512, 1024),               # a whole round, then 8 whole tiles (eight k stages)
    ([63], 64, 64),                          # one k stage
    ([65, 5], 192, 320),                     # three k stages
])
def test_linear_against_torch(lens, h_in, h_out):
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
        space = torch.empty(T * h_out, dtype=torch.float32, device="cuda")
        ref = x.double() @ wt.double().t()
        for g, s in enumerate(slot):
            if s >= 0:
                a, b = int(off[g]), int(off[g + 1])
                ref[a:b] += 2.0 * (0.5 + s) * (x[a:b].double() @ A[s].double()) @ Bm[s].double()
        for _ in range(3):  # the counts of split tiles are back at zero after every launch
            y = torch.full((T, h_out), float("nan"), dtype=torch.bfloat16, device="cuda")
            B.check(B.lora_linear_plan(pool.handle, plan, 0, 0, x.data_ptr(), wt.data_ptr(), y.data_ptr(), 2.0,
                                       torch.cuda.current_stream().cuda_stream, space.data_ptr(), space.numel() * 4))
            pool.check_fault()
            err, rms = (y.double() - ref).abs(), ref.pow(2).mean().sqrt()
            # one rounding of the output (half an ulp: 2^-9 of the element's binade, at most 2^-8 of its value) beside the
            # rounding of s.v to bf16 (2^-9 of each of its entries: well under 2^-8 of the RMS in the sum)
            assert bool((err <= 2.0**-8 * ref.abs() + 2.0**-7 * rms).all()), float((err / rms).max())
            assert float((y.double() - ref).norm() / ref.norm()) < 4e-3
    finally:
        pool.close()


def test_split_products_of_two_caches_at_the_same_time():
    """64 tiles in four parts each: one such launch fills the chip with parts of split tiles, two side by side get their places
    in whatever order, and whichever part of a tile comes last finishes it.  The results are those of one launch after
    the other, bit for bit."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    h_in, h, T, rank, n = 12288, 4096, 1000, 16, 12
    gen = torch.Generator(device="cuda").manual_seed(7)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    A, Bm = normal(h_in, rank, sigma=0.02).cpu(), normal(rank, h, sigma=0.02).cpu()
    x, wt = [normal(T, h_in) for _ in range(2)], [normal(h, h_in, sigma=0.02) for _ in range(2)]
    y = [[torch.empty(T, h, dtype=torch.bfloat16, device="cuda") for _ in range(n)] for _ in range(2)]
    pools = [LoraPool([(h_in, h)], 1, [rank], [1], B.LORA_BF16, max_tokens=T, max_segments=1) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    try:
        plans = []
        for q in pools:
            q.fill(0, 1, rank, 1.0, 0, 0, A, Bm)
            plans.append(q.plan(T, np.asarray([0, T], np.int32), np.zeros(1, np.int32), np.full(1, rank, np.int32)))
        torch.cuda.synchronize()

        def product(c, i, stream):
            B.check(B.lora_linear_plan(pools[c].handle, plans[c], 0, 0, x[c].data_ptr(), wt[c].data_ptr(), y[c][i].data_ptr(), 2.0, stream.cuda_stream))

        want = []
        for c in range(2):
            product(c, 0, streams[c])
            torch.cuda.synchronize()
            want.append(y[c][0].clone())
            y[c][0].zero_()
        torch.cuda.synchronize()
        for i in range(n):
            for c in range(2):
                product(c, i, streams[c])
        torch.cuda.synchronize()
        for c in range(2):
            pools[c].check_fault(streams[c])
            for i in range(n):
                assert torch.equal(y[c][i], want[c]), (c, i)
    finally:
        for q in pools:
            q.close()
