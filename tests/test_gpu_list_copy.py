"""Plans whose lists travel with their first launch: on other streams than the plan's, captured, followed at once by other plans and other streams, and where the first launch cannot take
them along."""
import numpy as np
import pytest
import torch

from streams import Busy

pytestmark = pytest.mark.gpu
H, N_L = 512, 6


class Batch:
    """A pool of 9 adapters, and batches of one-token requests (and a short prompt) over them."""

    def __init__(self, dtype="bf16", n_plans=2, flags=0, extra=()):
        from paper_2411_17741_amd import binding as B
        from paper_2411_17741_amd.pool import LoraPool

        self.B, self.dt = B, torch.bfloat16 if dtype == "bf16" else torch.float32
        self.ranks = [8, 16, 5, 64, 128, 33, 8, 100, 24]
        gen = torch.Generator(device="cuda").manual_seed(3)
        self.normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).to(self.dt)
        self.pool = LoraPool([(H, H)] + list(extra), N_L, [128], [9], B.LORA_BF16 if dtype == "bf16" else B.LORA_F32, max_tokens=256, max_segments=256, n_plans=n_plans, flags=flags)
        self.A, self.Bm = [self.normal(H, r, sigma=0.05) for r in self.ranks], [self.normal(r, H, sigma=0.05) for r in self.ranks]
        for layer in range(N_L):
            for i, r in enumerate(self.ranks):
                self.pool.fill(i, i + 1, r, 1.0, layer, 0, self.A[i].cpu(), self.Bm[i].cpu())
        torch.cuda.synchronize()
        self.x = self.normal(256, H)

    def segs(self, slots):
        slots = np.asarray(slots, np.int32)
        return len(slots), np.arange(len(slots) + 1, dtype=np.int32), slots, np.asarray(self.ranks, np.int32)[slots]

    def expect(self, base, slots, times=1):
        y = base.double().clone()
        for t, s in enumerate(slots):
            for _ in range(times):
                y[t] += 2.0 * (self.x[t].double() @ self.A[s].double()) @ self.Bm[s].double()
        return y

    def close_to(self, y, ref, times=1):
        # every pass rounds the output once and s.v once: 2^-8 of values of the size of the result and a little above
        rel = float((y.double() - ref).norm() / ref.norm())
        assert rel < (4e-3 * times if self.dt == torch.bfloat16 else 1e-5), rel


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_plans_in_a_row(dtype):
    """Plan after plan, each applied on a stream of its own and then at once on another one, there with the fixed scratch (two calls with the pool's would have to be ordered); a destroyed
    plan's memory goes to the next but one."""
    b = Batch(dtype)
    try:
        s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
        rng = np.random.default_rng(1)
        done = []
        torch.cuda.synchronize()
        for i in range(40):
            slots = rng.integers(0, 9, rng.integers(1, 60))
            base = b.normal(len(slots), H)
            y1, y2 = base.clone(), base.clone()
            torch.cuda.synchronize()
            plan = b.pool.plan(*b.segs(slots), stream=s1 if i % 3 == 0 else None)
            x = b.x[: len(slots)].contiguous()
            b.pool.apply_plan(plan, i % N_L, 0, x, y1, 2.0, stream=s1 if i % 2 else s2)
            b.B.check(b.B.lora_apply_plan_static(b.pool.handle, plan, (i + 1) % N_L, 0, x.data_ptr(), y2.data_ptr(), 2.0, (s2 if i % 2 else s1).cuda_stream))
            b.pool.plan_destroy(plan)
            done.append((x, y1, y2, base, slots))
        torch.cuda.synchronize()
        b.pool.check_fault()
        for _x, y1, y2, base, slots in done:
            ref = b.expect(base, slots)
            b.close_to(y1, ref)
            assert torch.equal(y1, y2)
    finally:
        b.pool.close()


@pytest.mark.parametrize("n_list", [1, 6, 24])
def test_first_use_as_a_list(n_list):
    """One projection, a list that takes the lists along, one of more wavefronts than read them over the link."""
    b = Batch()
    try:
        slots = np.arange(200 if n_list == 24 else 30) % 9
        base = b.normal(len(slots), H)
        x = b.x[: len(slots)].contiguous()
        for _ in range(3):
            plan = b.pool.plan(*b.segs(slots))
            y = [base.clone() for _ in range(n_list)]
            descs = b.B.make_descs([(i % N_L, 0, x.data_ptr(), y[i].data_ptr()) for i in range(n_list)])
            b.B.check(b.B.lora_apply_plan_multi(b.pool.handle, plan, descs, 2.0, torch.cuda.current_stream().cuda_stream))
            b.pool.apply_plan(plan, 0, 0, x, y[0], 2.0)  # out of the copied lists
            b.pool.plan_destroy(plan)
            b.close_to(y[0], b.expect(base, slots, 2), 2)
            ref = b.expect(base, slots)
            for t in y[1:]:
                b.close_to(t, ref)
        b.pool.check_fault()
    finally:
        b.pool.close()


@pytest.mark.parametrize("used", [False, True])
@pytest.mark.parametrize("n_plans", [1, 2])
def test_captured(used, n_plans):
    """A plan first used in a capture (its lists are then no part of the graph), or in an eager call before; replays with other plans' work in between."""
    b = Batch(n_plans=n_plans)
    try:
        slots, other = np.arange(40) % 9, (np.arange(25) * 4) % 9
        base = b.normal(40, H)
        x, y = b.x[:40].contiguous(), base.clone()
        plan = b.pool.plan(*b.segs(slots))
        if used:
            b.pool.apply_plan(plan, 1, 0, x, base.clone(), 2.0)
        stream = torch.cuda.Stream()
        graph = torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            b.pool.apply_plan(plan, 0, 0, x, y, 2.0, stream=stream)
        for i in range(4):
            y.copy_(base)
            if n_plans > 1 and i % 2:
                yo = b.normal(25, H)
                p2 = b.pool.plan(*b.segs(other))
                b.pool.apply_plan(p2, 0, 0, b.x[:25].contiguous(), yo, 2.0)
                b.pool.plan_destroy(p2)
            graph.replay()
            torch.cuda.synchronize()
            b.close_to(y, b.expect(base, slots))
        b.pool.check_fault()
    finally:
        b.pool.close()


def test_other_first_uses():
    """First used by a base product, with fencing off, in a cache without a side stream, and dumped before and after its first use."""
    for flags in (0, None):
        b = Batch(flags=0 if flags == 0 else __import__("paper_2411_17741_amd.binding", fromlist=["x"]).LORA_CACHE_NO_OVERLAP)
        try:
            slots = np.arange(50) % 9
            x, base = b.x[:50].contiguous(), b.normal(50, H)
            W = b.normal(H, H, sigma=0.05)
            plan = b.pool.plan(*b.segs(slots))
            rc, before, toks = b.B.lora_plan_dump(b.pool.handle, plan, 0)
            y = torch.empty_like(base)
            space = torch.empty(50 * H, dtype=torch.float32, device="cuda")
            b.B.check(b.B.lora_linear_plan(b.pool.handle, plan, 0, 0, x.data_ptr(), W.data_ptr(), y.data_ptr(), 2.0, torch.cuda.current_stream().cuda_stream, space.data_ptr(), space.numel() * 4))
            ref = b.expect((x.double() @ W.double().T), slots)
            b.close_to(y, ref)
            b.pool.plan_destroy(plan)
            plan = b.pool.plan(*b.segs(slots))
            b.B.check(b.B.lora_cache_set_fencing(b.pool.handle, 0))
            y = base.clone()
            b.pool.apply_plan(plan, 0, 0, x, y, 2.0)
            b.B.check(b.B.lora_cache_set_fencing(b.pool.handle, 1))
            b.close_to(y, b.expect(base, slots))
            b.pool.plan_destroy(plan)
            plan = b.pool.plan(*b.segs(slots))
            y = base.clone()
            b.pool.apply_plan(plan, 0, 0, x, y, 2.0)
            rc, after, toks2 = b.B.lora_plan_dump(b.pool.handle, plan, 0)
            assert np.array_equal(before, after) and np.array_equal(toks, toks2)
            b.close_to(y, b.expect(base, slots))
            b.pool.check_fault()
        finally:
            b.pool.close()


@pytest.mark.parametrize("small", [False, True])  # the run table's kernel where there are no panels
@pytest.mark.parametrize("lens", [[16], [70, 200, 33], [900, 1, 1, 640, 17]])  # units of 16 tokens; with tokens that are no tiles; panels or the run table
@pytest.mark.parametrize("first", ["apply", "list", "linear", "static", "captured"])
def test_plans_with_tiles(first, lens, small):
    """A plan with tiles: its lists travel with the tile shrink that is its first launch; everything behind it reads the copy."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    ranks, n, T, n_layers = [64, 128, 8, 33, 16], len(lens), sum(lens), 3
    gen = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    A, Bm = [normal(H, r, sigma=0.05) for r in ranks], [normal(r, H, sigma=0.05) for r in ranks]
    x, base, W = normal(T, H), normal(T, H), normal(H, H, sigma=0.05)
    pool = LoraPool([(H, H)], n_layers, [128], [5], B.LORA_BF16, max_tokens=T, max_segments=n, mfma_min_tokens=8, flags=B.LORA_CACHE_SMALL_SCRATCH if small else 0)
    try:
        for layer in range(n_layers):
            for i, r in enumerate(ranks):
                pool.fill(i, i + 1, r, 1.0, layer, 0, A[i].cpu(), Bm[i].cpu())
        delta = torch.zeros(T, H, dtype=torch.float64, device="cuda")
        for i in range(n):
            a, b = int(off[i]), int(off[i + 1])
            delta[a:b] = 2.0 * (x[a:b].double() @ A[i].double()) @ Bm[i].double()
        st = torch.cuda.current_stream().cuda_stream
        space = torch.empty(T * H, dtype=torch.float32, device="cuda")
        plans = []
        for turn in range(3):  # (the third plan lies where the first lay)
            plan = pool.plan(T, off, np.arange(n, dtype=np.int32), np.asarray(ranks[:n], np.int32))
            out = [base.clone() for _ in range(n_layers)]
            ref = [base.double() + delta] * n_layers

            def use(how):
                if how == "apply":
                    pool.apply_plan(plan, 0, 0, x, out[0], 2.0)
                elif how == "static":
                    B.check(B.lora_apply_plan_static(pool.handle, plan, 0, 0, x.data_ptr(), out[0].data_ptr(), 2.0, st))
                elif how == "list":
                    B.check(B.lora_apply_plan_multi(pool.handle, plan, B.make_descs([(l, 0, x.data_ptr(), out[l].data_ptr()) for l in range(n_layers)]), 2.0, st))
                else:
                    B.check(B.lora_linear_plan(pool.handle, plan, 0, 0, x.data_ptr(), W.data_ptr(), out[0].data_ptr(), 2.0, st, space.data_ptr(), space.numel() * 4))

            if first == "captured":
                graph, stream = torch.cuda.CUDAGraph(), torch.cuda.Stream()
                torch.cuda.synchronize()
                with torch.cuda.graph(graph, stream=stream):
                    pool.apply_plan(plan, 0, 0, x, out[0], 2.0, stream=stream)
                for _ in range(3):
                    out[0].copy_(base)
                    graph.replay()
                    torch.cuda.synchronize()
            else:
                use(first)
            count = n_layers if first == "list" else 1
            if first == "linear":
                ref = [x.double() @ W.double().T + delta]
            for y, r in zip(out[:count], ref):
                rel = float((y.double() - r).norm() / r.norm())
                assert rel < 4e-3, (turn, rel)  # the rounding of the output and of s.v, 2^-9 each on the mean and more
            again = [y.clone() for y in out]
            for y in out:
                y.copy_(base)
            use("apply" if first == "captured" else first)  # out of the copied lists: the same bits
            for y, z in zip(out[:count], again):
                assert torch.equal(y, z)
            if len(plans) == 1:
                pool.plan_destroy(plans.pop())
            plans.append(plan)
        pool.check_fault()
    finally:
        pool.close()


def test_one_call_with_tiles():
    """lora_apply on batches with tiles, call after call with nothing in between: its plans' memory goes round every four calls."""
    b = Batch()
    try:
        rng = np.random.default_rng(5)
        done = []
        for i in range(14):
            lens = rng.integers(1, 90, rng.integers(1, 4))
            slot = rng.permutation(9)[: len(lens)].astype(np.int32)
            T = int(lens.sum())
            x, base = b.x[:T].contiguous(), b.normal(T, H)
            y = base.clone()
            off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
            b.pool.apply(i % N_L, 0, x, y, off, slot, np.asarray(b.ranks, np.int32)[slot], 2.0)
            done.append((y, base, np.repeat(slot, lens)))
        torch.cuda.synchronize()
        b.pool.check_fault()
        for y, base, slots in done:
            b.close_to(y, b.expect(base, slots))
    finally:
        b.pool.close()


def test_two_plans_in_one_capture():
    """Two plans first used in one capture, the first by a batch whose GEMV launch is forked to the side stream (4 GB of tile tokens' activations and outputs and more), which is in
    the capture from then on; the second plan called before any replay, and replays beside eager calls."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    h, n_layers, prompt, rank = 8192, 32, 2700, 16
    assert prompt * 2 * n_layers * 3 * h >= 4e9
    gen = torch.Generator(device="cuda").manual_seed(9)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    T = prompt + 4
    pool = LoraPool([(h, h)], n_layers, [rank], [3], B.LORA_BF16, max_tokens=T, max_segments=8, n_plans=4)
    try:
        A, Bm = [normal(h, rank, sigma=0.02) for _ in range(3)], [normal(rank, h, sigma=0.05) for _ in range(3)]
        for i in range(3):
            a, b = A[i].cpu(), Bm[i].cpu()
            for layer in range(n_layers):
                pool.fill(i, i + 1, rank, 1.0, layer, 0, a, b)
        x = normal(T, h)
        large, small = torch.zeros(n_layers, T, h, dtype=torch.bfloat16, device="cuda"), torch.zeros(5, h, dtype=torch.bfloat16, device="cuda")
        torch.cuda.synchronize()
        p1 = pool.plan(T, [0, prompt, T - 3, T - 2, T - 1, T], [0, 1, 2, 1, 2], [rank] * 5)
        p2 = pool.plan(5, [0, 1, 2, 3, 4, 5], [2, 1, 0, 2, 1], [rank] * 5)
        descs = B.make_descs([(layer, 0, x.data_ptr(), large[layer].data_ptr()) for layer in range(n_layers)])

        def go(st, which=3):
            if which & 1:
                B.check(B.lora_apply_plan_multi(pool.handle, p1, descs, 2.0, st))
            if which & 2:
                pool.apply_plan(p2, 3, 0, x[:5], small, 2.0, stream=torch.cuda.ExternalStream(st) if st else None)

        stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(stream):
            graph.capture_begin(capture_error_mode="thread_local")
            go(stream.cuda_stream)
            graph.capture_end()
        now = torch.cuda.current_stream().cuda_stream
        go(now, 2)  # (before any replay)
        torch.cuda.synchronize()
        ref = torch.stack([2.0 * (x[t].double() @ A[s].double()) @ Bm[s].double() for t, s in enumerate([2, 1, 0, 2, 1])])
        assert float((small.double() - ref).norm() / ref.norm()) < 4e-3  # the roundings of the output and of s.v
        want_small = small.clone()
        for i in range(3):
            large.zero_(), small.zero_()
            graph.replay()
            torch.cuda.synchronize()
            if i == 0:
                got = large.clone()
            assert torch.equal(small, want_small) and torch.equal(large, got)
            small.zero_()
            go(now, 2)
            torch.cuda.synchronize()
            assert torch.equal(small, want_small)
        large.zero_()
        go(now, 1)
        torch.cuda.synchronize()
        pool.check_fault()
        assert torch.equal(large, got)  # captured and eager: the same bits
        B.lora_cache_set_timing(pool.handle, 1)
        go(now, 1)
        torch.cuda.synchronize()
        rc, t = B.lora_cache_read_timing(pool.handle)
        assert rc == B.LORA_OK and t["mfma_expand"][1] == 1 and t["gemv_fused"][1] >= 1, t  # one batch of them all
        for layer in (0, n_layers - 1):
            for t0, t1, s in ((0, prompt, 0), (prompt, T - 3, 1), (T - 3, T - 2, 2)):
                r = 2.0 * (x[t0:t1].double() @ A[s].double()) @ Bm[s].double()
                assert float((got[layer, t0:t1].double() - r).norm() / r.norm()) < 4e-3
    finally:
        pool.close()


@pytest.mark.parametrize("held", [1, 3])
def test_the_only_free_plan(held):
    """All plans but one are held: making that one again and again does not wait for the calls that used it last."""
    b = Batch(n_plans=held + 1)
    try:
        keep = [b.pool.plan(*b.segs([i])) for i in range(held)]
        busy, stream = torch.randn(4096, 4096, device="cuda"), torch.cuda.Stream()
        out = []
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            for i in range(3):
                slots = (np.arange(20 + i) * (i + 1)) % 9
                base = b.normal(len(slots), H)
                x, y = b.x[: len(slots)].contiguous(), base.clone()
                plan = b.pool.plan(*b.segs(slots))
                if i == 0:  # (its upload is not behind this)
                    for _ in range(60):
                        busy @ busy
                b.pool.apply_plan(plan, 0, 0, x, y, 2.0)
                b.pool.plan_destroy(plan)
                out.append((x, y, base, slots))
                if i == 0:
                    plan = b.pool.plan(*b.segs(slots))
                    assert not stream.query()  # the call is still to come
                    b.pool.plan_destroy(plan)
        torch.cuda.synchronize()
        b.pool.check_fault()
        for _x, y, base, slots in out:
            b.close_to(y, b.expect(base, slots))
        for i, plan in enumerate(keep):
            base = b.normal(1, H)
            y = base.clone()
            b.pool.apply_plan(plan, 1, 0, b.x[:1].contiguous(), y, 2.0)
            b.close_to(y, b.expect(base, [i]))
    finally:
        b.pool.close()


@pytest.mark.parametrize("how", ["captured", "static"])
def test_memory_that_a_graph_reads(how):
    """A graph's replay is still to come on the stream that the plan's memory is made anew on; the new plan is first used on another stream, by a capture or with scratch of its own."""
    b = Batch(n_plans=3)
    try:
        slots, other = np.arange(40) % 9, (np.arange(37) * 5 + 1) % 9
        x, busy = b.x[:40].contiguous(), torch.randn(4096, 4096, device="cuda")
        base, base2 = b.normal(40, H), b.normal(37, H)
        y, y2 = base.clone(), base2.clone()
        s1, s2, graph, graph2 = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
        torch.cuda.synchronize()
        plan = b.pool.plan(*b.segs(slots), stream=s1)
        with torch.cuda.graph(graph, stream=s1):
            b.pool.apply_plan(plan, 0, 0, x, y, 2.0, stream=s1)
        torch.cuda.synchronize()
        with torch.cuda.stream(s1):
            for _ in range(60):
                busy @ busy
            graph.replay()
        b.pool.plan_destroy(plan)
        for _ in range(2):  # the other two
            b.pool.plan_destroy(b.pool.plan(*b.segs(slots), stream=s1))
        plan2 = b.pool.plan(*b.segs(other), stream=s1)
        assert plan2.value == plan.value and not s1.query()
        if how == "captured":
            with torch.cuda.stream(s2):
                graph2.capture_begin(capture_error_mode="thread_local")
                b.pool.apply_plan(plan2, 1, 0, x[:37], y2, 2.0, stream=s2)
                graph2.capture_end()
                graph2.replay()
        else:
            b.B.check(b.B.lora_apply_plan_static(b.pool.handle, plan2, 1, 0, x.data_ptr(), y2.data_ptr(), 2.0, s2.cuda_stream))
        torch.cuda.synchronize()
        b.pool.check_fault()
        b.close_to(y, b.expect(base, slots))
        b.close_to(y2, b.expect(base2, other))
    finally:
        b.pool.close()


@pytest.mark.parametrize("n_plans", [1, 2])  # the new lists uploaded; copied by a launch
def test_a_call_with_fixed_scratch_still_to_come(n_plans):
    """A plan's latest call is over, one before it with scratch of its own is still to come on another stream: the next plan in its memory leaves it its lists."""
    b = Batch(n_plans=n_plans)
    try:
        slots, other = np.arange(40) % 9, (np.arange(37) * 5 + 1) % 9
        x, busy = b.x[:40].contiguous(), Busy()
        base = b.normal(40, H)
        y = [base.clone() for _ in range(4)]
        s1, s2 = busy.one, busy.two
        plan = b.pool.plan(*b.segs(slots), stream=s2)
        torch.cuda.synchronize()
        b.pool.apply_plan(plan, 0, 0, x, y[0], 2.0, stream=s2)
        torch.cuda.synchronize()
        busy.start()
        b.B.check(b.B.lora_apply_plan_static(b.pool.handle, plan, 1, 0, x.data_ptr(), y[1].data_ptr(), 2.0, s1.cuda_stream))
        b.pool.apply_plan(plan, 2, 0, x, y[2], 2.0, stream=s2)
        s2.synchronize()
        b.pool.plan_destroy(plan)
        for _ in range(n_plans - 1):
            b.pool.plan_destroy(b.pool.plan(*b.segs(slots), stream=s2))
        again = b.pool.plan(*b.segs(other), stream=s2)
        assert again.value == plan.value and not s1.query()
        b.pool.apply_plan(again, 3, 0, x[:37], y[3][:37], 2.0, stream=s2)
        torch.cuda.synchronize()
        b.pool.check_fault()
        for i in range(3):
            b.close_to(y[i], b.expect(base, slots))
        b.close_to(y[3][:37], b.expect(base[:37], other))
    finally:
        b.pool.close()


@pytest.mark.parametrize("why,lens", [("own stream", [1] * 50), ("own stream", [200, 56]), ("split", [1] * 50)])
def test_lists_made_ahead_on_another_stream(why, lens):
    """Plans made on a stream without applies, and lists that no launch can take along: uploaded on the stream of lora_plan_create, which calls on other streams wait for."""
    from paper_2411_17741_amd import binding as B

    b = Batch(flags=B.LORA_CACHE_SPLIT_GEMV if why == "split" else 0)
    try:
        T, n = sum(lens), len(lens)
        slot = (np.arange(n) % 9).astype(np.int32)
        segs = T, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), slot, np.asarray(b.ranks, np.int32)[slot]
        x, base, busy = b.x[:T].contiguous(), b.normal(T, H), Busy()
        y, y0, done = base.clone(), base.clone(), torch.cuda.Event()
        s1, s2 = busy.one, busy.two
        torch.cuda.synchronize()
        if why == "own stream":
            plan = b.pool.plan(*segs, stream=s2)
            b.pool.apply_plan(plan, 0, 0, x, y0, 2.0, stream=s2)
            b.pool.plan_destroy(plan)
            torch.cuda.synchronize()
        busy.start()
        done.record(s1)
        plan = b.pool.plan(*segs, stream=s1)
        b.pool.apply_plan(plan, 1, 0, x, y, 2.0, stream=s2)
        assert not done.query()
        s2.synchronize()
        assert done.query()
        torch.cuda.synchronize()
        b.pool.check_fault()
        b.close_to(y, b.expect(base, np.repeat(slot, lens)))
    finally:
        b.pool.close()


@pytest.mark.parametrize("lens", [[1] * 50, [200, 56]])
@pytest.mark.parametrize("one_call", [False, True])
def test_an_error_of_an_earlier_call(lens, one_call):
    """An error that another call of the thread has left behind is what the launch that takes the lists along returns, though it is on its way: it is over when the call returns, nothing
    guards the host's copy of the lists from then on; the plan stays usable."""
    b = Batch()
    try:
        T, n = sum(lens), len(lens)
        slot = (np.arange(n) % 9).astype(np.int32)
        segs = T, np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), slot, np.asarray(b.ranks, np.int32)[slot]
        x, base, busy = b.x[:T].contiguous(), b.normal(T, H), torch.randn(4096, 4096, device="cuda")
        y, stream = base.clone(), torch.cuda.Stream()
        torch.cuda.synchronize()
        plan = b.pool.plan(*segs, stream=stream)
        with torch.cuda.stream(stream):
            for _ in range(60):
                busy @ busy
        assert b.B._lib.hipSetDevice(9999) != 0  # no such device
        if one_call:
            rc = b.B.lora_apply(b.pool.handle, 0, 0, x.data_ptr(), y.data_ptr(), T, *segs[1:], 2.0, stream.cuda_stream)
        else:
            rc = b.B.lora_apply_plan(b.pool.handle, plan, 0, 0, x.data_ptr(), y.data_ptr(), 2.0, stream.cuda_stream)
        assert rc == b.B.LORA_E_HIP
        assert stream.query()
        for _ in range(2):
            y.copy_(base)
            b.pool.apply_plan(plan, 0, 0, x, y, 2.0)
            b.close_to(y, b.expect(base, np.repeat(slot, lens)))
            b.pool.plan_destroy(plan)
            plan = b.pool.plan(*segs)
        b.pool.check_fault()
    finally:
        b.pool.close()


@pytest.mark.parametrize("lens", [[1] * 50, [200, 56]])
def test_a_copying_launch_still_to_come(lens):
    """The launch that takes the lists along is still to come: a call on another stream waits for it, and so does the plan that is made in that memory next."""
    b = Batch()
    try:
        T, n = sum(lens), len(lens)
        x, base, busy = b.x[:T].contiguous(), b.normal(T, H), Busy()
        y, early = [base.clone() for _ in range(6)], torch.cuda.Event()
        s1, s2 = busy.one, busy.two
        slots = [((np.arange(n) * (i + 1) + i) % 9).astype(np.int32) for i in range(5)]
        off, ranks = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), np.asarray(b.ranks, np.int32)

        def make(i):
            return b.pool.plan(T, off, slots[i], ranks[slots[i]], stream=s1)

        torch.cuda.synchronize()
        plan = make(0)
        b.pool.apply_plan(plan, 0, 0, x, y[0], 2.0, stream=s1)  # (from here on s1 is a stream with applies)
        b.pool.plan_destroy(plan)
        torch.cuda.synchronize()

        busy.start()
        plan = make(1)
        b.pool.apply_plan(plan, 1, 0, x, y[1], 2.0, stream=s2)
        s2.synchronize()
        assert not s1.query()  # nothing of the plan is behind the work on s1: its lists travelled
        b.pool.plan_destroy(plan)
        torch.cuda.synchronize()

        busy.start()
        early.record(s1)
        plan = first = make(2)
        b.pool.apply_plan(plan, 2, 0, x, y[2], 2.0, stream=s1)
        b.B.check(b.B.lora_apply_plan_static(b.pool.handle, plan, 3, 0, x.data_ptr(), y[3].data_ptr(), 2.0, s2.cuda_stream))
        b.pool.plan_destroy(plan)
        plan = make(3)
        b.pool.apply_plan(plan, 4, 0, x, y[4], 2.0, stream=s1)
        b.pool.plan_destroy(plan)
        assert not early.query()
        plan = make(4)
        assert early.query()  # waited for the call that read the lists with the host
        assert plan.value == first.value
        b.pool.apply_plan(plan, 5, 0, x, y[5], 2.0, stream=s1)
        torch.cuda.synchronize()
        b.pool.check_fault()
        for i, k in enumerate([0, 1, 2, 2, 3, 4]):
            b.close_to(y[i], b.expect(base, np.repeat(slots[k], lens)))
    finally:
        b.pool.close()


@pytest.mark.parametrize("h_in,length,travel", [(128, 2000, True), (128, 2100, False), (512, 2100, True)])  # 1500 blocks; 1584; 1584, and panels on more projections
def test_tile_shrinks_of_many_blocks(h_in, length, travel):
    """Lists travel with a tile shrink whose blocks take 16 tokens and 16 rank rows each up to 1536 of them; where no list of projections makes another launch they are uploaded on the stream that made the plan."""
    from paper_2411_17741_amd import binding as B
    from paper_2411_17741_amd.pool import LoraPool

    rank, T, h_out = 96, 2 * length, 128
    gen = torch.Generator(device="cuda").manual_seed(length)
    normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
    A, Bm = [normal(h_in, rank, sigma=0.05) for _ in range(2)], [normal(rank, h_out, sigma=0.05) for _ in range(2)]
    segs = T, np.asarray([0, length, T], np.int32), np.arange(2, dtype=np.int32), np.full(2, rank, np.int32)
    pool = LoraPool([(h_in, h_out)], 2, [128], [2], B.LORA_BF16, max_tokens=T, max_segments=2, mfma_min_tokens=8)
    try:
        for layer in range(2):
            for i in range(2):
                pool.fill(i, i + 1, rank, 1.0, layer, 0, A[i].cpu(), Bm[i].cpu())
        x, base, busy, done = normal(T, h_in), normal(T, h_out), Busy(), torch.cuda.Event()
        y, (s1, s2) = [base.clone() for _ in range(2)], (busy.one, busy.two)
        torch.cuda.synchronize()
        plan = pool.plan(*segs, stream=s1)
        rc, units, _toks = B.lora_plan_dump(pool.handle, plan, 0)
        assert rc == B.LORA_OK and int((units["kind"] == B.LORA_UNIT_DIRECT_SHRINK).sum()) == 2 * -(-length // 16) * rank // 16
        pool.apply_plan(plan, 0, 0, x, y[0], 2.0, stream=s1)  # (from here on s1 is a stream with applies)
        pool.plan_destroy(plan)
        torch.cuda.synchronize()
        busy.start()
        done.record(s1)
        plan = pool.plan(*segs, stream=s1)
        pool.apply_plan(plan, 1, 0, x, y[1], 2.0, stream=s2)
        s2.synchronize()
        assert done.query() != travel  # uploaded behind the work on s1, or nothing of the plan is there
        torch.cuda.synchronize()
        pool.check_fault()
        for out in y:
            for i in range(2):
                rows = slice(i * length, (i + 1) * length)
                ref = base[rows].double() + 2.0 * (x[rows].double() @ A[i].double()) @ Bm[i].double()
                assert float((out[rows].double() - ref).norm() / ref.norm()) < 4e-3  # the roundings of the output and of s.v
    finally:
        pool.close()
