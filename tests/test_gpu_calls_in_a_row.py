"""lora_apply calls back to back, each with a batch of its own: the lists of a call are read by its kernels where the host wrote them, and must not be
written over before that."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fencing", [1, 0])
@pytest.mark.parametrize("dtype,tokens", [("f32", 5), ("bf16", 3), ("bf16", 150), ("bf16", 1500)])  # 1500: past the limit of lists read in place
def test_applies_in_a_row(dtype, tokens, fencing):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    h, ranks, n = 512, [8, 16, 33, 128] * 4, 14
    gen = torch.Generator(device="cuda").manual_seed(tokens)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).to(dt)
    pool = LoraPool([(h, h)], 1, [128], [16], B.LORA_F32 if dtype == "f32" else B.LORA_BF16, max_tokens=tokens, max_segments=tokens, mfma_min_tokens=100000)
    try:
        for i, r in enumerate(ranks):
            pool.fill(i, i + 1, r, 1.0, 0, 0, normal(h, r, sigma=0.02).cpu(), normal(r, h, sigma=0.02).cpu())
        B.lora_cache_set_fencing(pool.handle, fencing)
        rng = np.random.default_rng(tokens)
        off = np.arange(tokens + 1, dtype=np.int32)
        slots = [rng.integers(0, 16, tokens).astype(np.int32) for _ in range(n)]
        x, base = normal(tokens, h), normal(tokens, h)
        rank_of = np.asarray(ranks, np.int32)
        want, got = [base.clone() for _ in range(n)], [base.clone() for _ in range(n)]
        for y, s in zip(want, slots):
            pool.apply(0, 0, x, y, off, s, rank_of[s], 2.0)
            torch.cuda.synchronize()
        streams = [torch.cuda.Stream(), torch.cuda.Stream()]
        busy = torch.randn(2048, 2048, device="cuda")
        torch.cuda.synchronize()
        for i, (y, s) in enumerate(zip(got, slots)):
            # in one stream's order, or (the hand-over words of a cache are one set) the second stream behind the first
            st = streams[i >= n // 2]
            if i == n // 2:
                streams[1].wait_stream(streams[0])
            with torch.cuda.stream(st):
                if i % 5 == 0:
                    busy @ busy  # the calls behind wait on the device while the host goes on
                pool.apply(0, 0, x, y, off, s, rank_of[s], 2.0)
        torch.cuda.synchronize()
        pool.check_fault()
        for i in range(n):
            assert torch.equal(got[i], want[i]), i
    finally:
        pool.close()
