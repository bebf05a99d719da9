"""lora_linear_plan where its grid can go wrong: tiles split along k into every number of parts (the sums of the parts of a
tile meet in its output), whole rounds before a split one, ragged panels, odd numbers of k stages."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,h_in,h_out", [
    ([300], 4096, 1024),                     # 8 tiles of 256 x 256: eight parts
    ([1000], 4160, 1280),                    # 20 to 25 tiles, 65 k stages: six or five parts
    ([1, 700, 900, 2, 833], 2112, 1024),     # 44 tiles, 33 k stages: three parts
    ([4000, 100], 4096, 1088),               # 85 tiles, the last column panel 64 wide: three parts
    ([3100], 2048, 2432),                    # 130 tiles: whole
    ([2000, 17], 4096, 4096),                # 128 to 144 tiles: two parts or whole
    ([16384, 190], 512, 1024),               # a whole round, then a few tiles in two parts (eight k stages)
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
