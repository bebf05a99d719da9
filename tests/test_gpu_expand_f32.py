"""The fp32 expand at the edges of its passes, in launches of few wavefronts and of many: one to sixteen granules of 8 ranks, one to three blocks of 64 columns past a pass, an infinity in a weight
that no clamped load may bring into other columns."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h_out", [64, 320, 1024, 1088])
@pytest.mark.parametrize("ranks", [(8, 16, 32), (5, 24, 64), (40, 72, 128), (1, 100, 12), (48, 56, 96)])
@pytest.mark.parametrize("many", [False, True])
def test_f32_expand(ranks, h_out, many):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    h_in, lens = 128, [1, 7, 4]
    if many:  # 60 batches of four tokens, 32 shrink blocks of four wavefronts each
        lens, ranks = lens + [240], ranks + (128,)
    gen = torch.Generator(device="cuda").manual_seed(h_out + ranks[0])
    normal = lambda *s: torch.randn(*s, generator=gen, device="cuda")
    T, n = sum(lens), len(lens)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    A, Bm = [normal(h_in, r) for r in ranks], [normal(r, h_out) for r in ranks]
    Bm[1][-1, h_out - 1] = float("inf")
    x, base = normal(T, h_in), normal(T, h_out)
    pool = LoraPool([(h_in, h_out)], 1, [128], [n], B.LORA_F32, max_tokens=T, max_segments=n)
    try:
        for i in range(n):
            pool.fill(i, i + 1, ranks[i], 0.5 + i, 0, 0, A[i].cpu(), Bm[i].cpu())
        plan = pool.plan(T, off, np.arange(n, dtype=np.int32), np.asarray(ranks, np.int32))
        rc, info = B.lora_plan_info(plan)
        assert rc == B.LORA_OK and (4 * info.n_gemv_shrink_items > 7424) == many
        pool.plan_destroy(plan)
        y = base.clone()
        pool.apply(0, 0, x, y, off, np.arange(n, dtype=np.int32), np.asarray(ranks, np.int32), 2.0)
        pool.check_fault()
        for i in range(n):
            a, b = int(off[i]), int(off[i + 1])
            s = 2.0 * (0.5 + i)
            ref = base[a:b].double() + s * (x[a:b].double() @ A[i].double()) @ Bm[i].double()
            room = base[a:b].double().abs() + s * (x[a:b].double().abs() @ A[i].double().abs()) @ Bm[i].double().abs()
            cols = slice(0, h_out - 1) if i == 1 else slice(0, h_out)
            # sums of at most h_in + rank + 3 roundings of 2^-24 each, of terms whose absolute values add up to `room`
            assert bool(((y[a:b].double() - ref)[:, cols].abs() <= (h_in + ranks[i] + 3) * 2.0**-24 * room[:, cols]).all())
            assert i != 1 or not bool(torch.isfinite(y[a:b, h_out - 1]).any())
    finally:
        pool.close()
