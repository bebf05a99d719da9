"""Whole adapters through the staging buffers: however the host arrays lie, the slot's slabs hold the adapter's values
in their layout (At [rs][h_in], Bp [rs/8][h_out][8], rows past the rank zero), bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _slab(A, Bm, rs):
    (h_in, r), h_out = A.shape, Bm.shape[1]
    At, Bp = torch.zeros(rs, h_in, dtype=A.dtype), torch.zeros(rs, h_out, dtype=A.dtype)
    At[:r], Bp[:r] = A.t(), Bm
    return torch.cat([At.flatten(), Bp.view(rs // 8, 8, h_out).permute(0, 2, 1).flatten()])


# more parts than a launch takes; more bytes than a buffer (16 MB) takes; one part; ranks that are no multiple of 8
@pytest.mark.parametrize("rank,layers,dtype", [(8, 33, "bf16"), (128, 40, "bf16"), (5, 1, "bf16"), (100, 3, "f32")])
@pytest.mark.parametrize("where", ["arena", "apart", "pageable"])
def test_staged_fill_of_a_whole_adapter(rank, layers, dtype, where):
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    proj = [(1024, 1088), (64, 192)]
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    pool = LoraPool(proj, layers, [rank], [2], B.LORA_BF16 if dtype == "bf16" else B.LORA_F32, max_tokens=1, max_segments=1)
    try:
        sizes = [s for _ in range(layers) for h_in, h_out in proj for s in (h_in * rank, rank * h_out)]
        arena = torch.randn(sum(sizes), generator=torch.Generator().manual_seed(rank)).to(dt)
        if where != "pageable":
            arena = arena.pin_memory()
        arrays = list(arena.split(sizes))
        if where == "apart":
            arrays = [a.clone().pin_memory() for a in arrays]
        entries = [(l, p, arrays[4 * l + 2 * p].data_ptr(), arrays[4 * l + 2 * p + 1].data_ptr()) for l in range(layers) for p in range(2)]
        entries = [(0, 0) + entries[-2][2:]] + entries  # the first part twice: the later one counts
        B.check(B.lora_cache_fill_slot_parts(pool.handle, 1, 7, rank, 1.0, B.make_fill_parts(entries), torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        rs = (rank + 7) // 8 * 8
        for l in range(layers):
            for p, (h_in, h_out) in enumerate(proj):
                _rc, at, _n = B.lora_cache_slab(pool.handle, l, p, 1)
                n = rs * (h_in + h_out) * arena.element_size()
                got = pool.buf[at - pool.buf.data_ptr():][:n].cpu().view(dt)
                a, b = arrays[4 * l + 2 * p], arrays[4 * l + 2 * p + 1]
                assert torch.equal(got, _slab(a.view(h_in, rank), b.view(rank, h_out), rs)), (l, p)
    finally:
        pool.close()
