"""The event that stands for the end of a call, as it rides on the call's last kernel: an upload into a plan's buffer and
a refill of a slot, both on another stream, wait for the applies that still read them."""
import numpy as np
import pytest
import torch

from streams import Busy

pytestmark = pytest.mark.gpu


# the last kernel is the GEMV launch; the tile expand; the join of a batch with both; a call that times its kernels
@pytest.mark.parametrize("lens,m0,timed", [([1] * 40, 0, False), ([512] * 40, 16, False), ([512, 1] * 20, 16, False), ([512] * 40, 16, True)])
def test_upload_and_refill_wait_for_applies_on_another_stream(lens, m0, timed):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    h, T, rank, n_calls = 2048, sum(lens), 64, 70  # more calls than the ring of fences holds
    gen = torch.Generator().manual_seed(len(lens) + m0)
    A, Bm = ([torch.randn(*s, generator=gen).mul_(0.02).bfloat16().pin_memory() for _ in range(3)] for s in ((h, rank), (rank, h)))
    x = torch.randn(T, h, generator=gen).bfloat16().cuda()
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    ranks = np.full(len(lens), rank, np.int32)
    outs = []
    for overlapped in (False, True):
        pool = LoraPool([(h, h)], 1, [rank], [2], B.LORA_BF16, max_tokens=T, max_segments=len(lens), n_plans=1, mfma_min_tokens=m0)
        try:
            for s in (0, 1):
                pool.fill(s, s + 1, rank, 1.0, 0, 0, A[s], Bm[s], pin=False)
            torch.cuda.synchronize()
            B.lora_cache_set_timing(pool.handle, int(timed))
            first, second = (torch.cuda.Stream(), torch.cuda.Stream()) if overlapped else (torch.cuda.current_stream(),) * 2
            y0, y1 = torch.zeros(T, h, dtype=torch.bfloat16, device="cuda"), torch.zeros(T, h, dtype=torch.bfloat16, device="cuda")
            torch.cuda.synchronize()
            plan = pool.plan(T, off, np.zeros(len(lens), np.int32), ranks, stream=first)
            for _ in range(n_calls):
                pool.apply_plan(plan, 0, 0, x, y0, 2.0, stream=first)
            pool.plan_destroy(plan)
            done = torch.cuda.Event()
            done.record(first)
            B.check(B.lora_cache_release_slot(pool.handle, 0))
            pool.fill(0, 3, rank, 1.0, 0, 0, A[2], Bm[2], stream=second, pin=False)  # waits for the applies of `first`
            plan = pool.plan(T, off, np.ones(len(lens), np.int32), ranks, stream=second)  # the same buffer
            second.wait_event(done)  # (applies of one cache share its scratch: the caller orders them)
            pool.apply_plan(plan, 0, 0, x, y1, 2.0, stream=second)
            pool.plan_destroy(plan)
            pool.check_fault(second)
            torch.cuda.synchronize()
            outs.append((y0, y1))
        finally:
            pool.close()
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    assert outs[0][0].abs().max() > 0 and outs[0][1].abs().max() > 0


def test_refill_waits_for_a_call_with_fixed_scratch_still_to_come():
    """The slot's latest apply is over, one before it with scratch of its own is still to come on another stream: a refill leaves it its weights."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    h, T, rank = 512, 24, 16
    gen = torch.Generator().manual_seed(4)
    A, Bm = ([torch.randn(*s, generator=gen).mul_(0.05).bfloat16().pin_memory() for _ in range(2)] for s in ((h, rank), (rank, h)))
    x = torch.randn(T, h, generator=gen).bfloat16().cuda()
    pool = LoraPool([(h, h)], 1, [rank], [1], B.LORA_BF16, max_tokens=T, max_segments=T, n_plans=1)
    try:
        pool.fill(0, 1, rank, 1.0, 0, 0, A[0], Bm[0], pin=False)
        y, busy, s3 = torch.zeros(4, T, h, dtype=torch.bfloat16, device="cuda"), Busy(), torch.cuda.Stream()
        s1, s2 = busy.one, busy.two
        plan = pool.plan(T, np.arange(T + 1), np.zeros(T, np.int32), np.full(T, rank, np.int32))
        torch.cuda.synchronize()
        busy.start()
        B.check(B.lora_apply_plan_static(pool.handle, plan, 0, 0, x.data_ptr(), y[0].data_ptr(), 2.0, s1.cuda_stream))
        pool.apply_plan(plan, 0, 0, x, y[1], 2.0, stream=s2)
        s2.synchronize()
        pool.plan_destroy(plan)
        B.check(B.lora_cache_release_slot(pool.handle, 0))
        assert not s1.query()
        pool.fill(0, 2, rank, 1.0, 0, 0, A[1], Bm[1], stream=s3, pin=False)
        torch.cuda.synchronize()
        plan = pool.plan(T, np.arange(T + 1), np.zeros(T, np.int32), np.full(T, rank, np.int32))
        pool.apply_plan(plan, 0, 0, x, y[2], 2.0)
        torch.cuda.synchronize()
        pool.check_fault()
        assert torch.equal(y[0], y[1]) and not torch.equal(y[0], y[2])
        for i, w in ((0, 0), (2, 1)):
            ref = 2.0 * (x.double() @ A[w].cuda().double()) @ Bm[w].cuda().double()
            assert float((y[i].double() - ref).norm() / ref.norm()) < 4e-3  # the roundings of the output and of s.v
    finally:
        pool.close()
