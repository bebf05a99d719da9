"""Plans whose calls for one projection leave everything to the GEMV kernels, in launches that take tiles: lists of many projections (more than a batch with tiles holds) and the base
product, called and captured."""
import numpy as np
import pytest
import torch

from plan_checks import check_plan_units
from streams import Busy

pytestmark = pytest.mark.gpu
RANKS = [16, 100, 5, 64]


class Case:
    def __init__(self, lens, h_in, h_out, n_layers, seed=0):
        from paper_2411_17741_amd import binding as B
        from paper_2411_17741_amd.pool import LoraPool

        self.B, self.T, self.n_layers, self.shape = B, sum(lens), n_layers, (h_in, h_out)
        self.off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
        self.slot = np.asarray([i % 4 if n > 1 else 4 + i % 12 for i, n in enumerate(lens)], np.int32)  # one-token requests: pools of a few
        gen = torch.Generator(device="cuda").manual_seed(seed)
        normal = lambda *s, sigma=1.0: torch.randn(*s, generator=gen, device="cuda").mul_(sigma).bfloat16()
        self.rank_of = np.asarray([RANKS[s % 4] for s in range(16)], np.int32)
        self.A, self.Bm = [normal(h_in, int(r), sigma=0.02) for r in self.rank_of], [normal(int(r), h_out, sigma=0.02) for r in self.rank_of]
        self.pool = LoraPool([(h_in, h_out)], n_layers, [128], [16], B.LORA_BF16, max_tokens=self.T, max_segments=len(lens))
        for s in range(16):
            a, b = self.A[s].cpu(), self.Bm[s].cpu()
            for layer in range(n_layers):
                self.pool.fill(s, s + 1, int(self.rank_of[s]), 0.5 + s / 4, layer, 0, a, b)
        self.x, self.base, self.wt = [normal(self.T, h_in) for _ in range(n_layers)], normal(n_layers, self.T, h_out), normal(h_out, h_in, sigma=0.02)
        self.plan = self.pool.plan(self.T, self.off, self.slot, self.rank_of[self.slot])
        rc, info = B.lora_plan_info(self.plan)
        assert rc == B.LORA_OK and info.n_tiles == 0  # a call for one projection: GEMV alone
        self.stream = torch.cuda.current_stream().cuda_stream

    def check(self, y, layer, base):
        at = torch.as_tensor(np.repeat(self.slot, np.diff(self.off)), device="cuda")
        ref, rounding = base.double().clone(), torch.zeros_like(base, dtype=torch.float64)
        for s in range(16):
            v = 2.0 * (0.5 + s / 4) * (self.x[layer][at == s].double() @ self.A[s].double())
            ref[at == s] += v @ self.Bm[s].double()
            rounding[at == s] = v.abs() @ self.Bm[s].double().abs()
        # the rounding of the output (2^-8 of its value) and that of every entry of s.v (2^-8 of its term); an eighth more for the sums in fp32
        assert bool(((y.double() - ref).abs() <= 1.125 * 2.0**-8 * (ref.abs() + rounding)).all())

    def kernels(self, call):
        """kinds of kernels that a call launches"""
        self.B.lora_cache_set_timing(self.pool.handle, 1)
        call()
        torch.cuda.synchronize()
        rc, t = self.B.lora_cache_read_timing(self.pool.handle)
        self.B.lora_cache_set_timing(self.pool.handle, 0)
        assert rc == self.B.LORA_OK
        return {k for k, (_ms, n) in t.items() if n}

    def apply_list(self, y, stream=None):
        B = self.B
        descs = B.make_descs([(layer, 0, self.x[layer].data_ptr(), y[layer].data_ptr()) for layer in range(self.n_layers)])
        B.check(B.lora_apply_plan_multi(self.pool.handle, self.plan, descs, 2.0, stream or self.stream))


LENS = [[77, 1, 1, 30, 1] + [1] * 20, [60, 41, 9, 130] + [1] * 12 * 9]  # the second: pools of nine one-token requests become tiles too


@pytest.mark.parametrize("lens", LENS)
@pytest.mark.parametrize("n_layers", [40, 64, 100])  # one batch with tiles, the most it holds, two of them
def test_lists(lens, n_layers):
    c = Case(lens, 512, 1024, n_layers)
    try:
        y = c.base.clone()
        kinds = c.kernels(lambda: c.apply_list(y))
        assert "mfma_expand" in kinds
        # what the kernels read, as the device holds it
        check_plan_units(c.pool.handle, c.plan, c.T, c.off, c.slot, c.rank_of[c.slot], [c.shape], {s: 0.5 + s / 4 for s in range(16)}, tiled=True)
        for layer in range(n_layers):
            c.check(y[layer], layer, c.base[layer])
        again = c.base.clone()
        c.apply_list(again)
        assert torch.equal(again, y)
        one = c.base[0].clone()
        assert c.kernels(lambda: c.pool.apply_plan(c.plan, 0, 0, c.x[0], one, 2.0)) == {"gemv_fused"}
        c.check(one, 0, c.base[0])
        # another batch in the same plan: nothing of the lists is left
        c.pool.plan_destroy(c.plan)
        c.plan = c.pool.plan(c.T, c.off, c.slot[::-1].copy() * 0, np.full(len(lens), RANKS[0], np.int32))
        c.slot = c.slot * 0
        z = c.base.clone()
        c.apply_list(z)
        c.pool.check_fault()
        c.check(z[n_layers - 1], n_layers - 1, c.base[n_layers - 1])
    finally:
        c.pool.close()


@pytest.mark.parametrize("lens", [[200, 90, 77], [400, 350, 90, 1, 1]])
@pytest.mark.parametrize("h_in,h_out", [(2048, 1024), (1088, 2112)])
def test_base_product(lens, h_in, h_out):
    c = Case(lens, h_in, h_out, 8)
    try:
        B, space = c.B, torch.empty(c.T * h_out, dtype=torch.float32, device="cuda")
        full = c.x[0].double() @ c.wt.double().t()
        for workspace in (True, False):
            outs = []
            for _ in range(2):
                y = torch.full((c.T, h_out), float("nan"), dtype=torch.bfloat16, device="cuda")
                call = lambda: B.check(B.lora_linear_plan(c.pool.handle, c.plan, 0, 0, c.x[0].data_ptr(), c.wt.data_ptr(), y.data_ptr(), 2.0, c.stream,
                                                          space.data_ptr() if workspace else 0, space.numel() * 4 if workspace else 0))
                kinds = c.kernels(call)
                assert "mfma_shrink" in kinds and "linear" in kinds
                outs.append(y)
            assert torch.equal(outs[0], outs[1])
            # (without a workspace the GEMV rows' term is rounded on its way: at most 2^-9 of it)
            at = torch.as_tensor(np.repeat(c.slot, np.diff(c.off)), device="cuda")
            ref, rounding = full.clone(), torch.zeros_like(full)
            for s in range(16):
                v = 2.0 * (0.5 + s / 4) * (c.x[0][at == s].double() @ c.A[s].double())
                ref[at == s] += v @ c.Bm[s].double()
                rounding[at == s] = v.abs() @ c.Bm[s].double().abs()
            assert bool(((y.double() - ref).abs() <= 1.125 * 2.0**-8 * (ref.abs() + 1.5 * rounding) + 2.0**-12 * full.abs().max()).all())
    finally:
        c.pool.close()


@pytest.mark.parametrize("first", ["capture", "eager"])
@pytest.mark.parametrize("call", ["list", "base product"])
def test_captured(call, first):
    """The same call gives the same bits, whether it is captured before any other, behind one, or not at all; every replay does."""
    product = call == "base product"
    c = Case([200, 90, 77], 2048, 1024, 8) if product else Case(LENS[0], 512, 1024, 40)
    try:
        B, space = c.B, torch.empty(c.T * 1024, dtype=torch.float32, device="cuda")

        def go(y):
            stream = torch.cuda.current_stream().cuda_stream
            if product:
                B.check(B.lora_linear_plan(c.pool.handle, c.plan, 0, 0, c.x[0].data_ptr(), c.wt.data_ptr(), y.data_ptr(), 2.0, stream, space.data_ptr(), space.numel() * 4))
            else:
                c.apply_list(y, stream)

        y = c.base.clone()
        eager = c.base.clone()
        if first == "eager":
            go(eager)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            go(y)
        outs = []
        for i in range(4):
            y.copy_(c.base)
            if i == 2 and first == "capture":
                go(eager)  # eager work in between
            graph.replay()
            torch.cuda.synchronize()
            outs.append(y.clone())
        c.pool.check_fault()
        for o in outs:
            assert torch.equal(o, eager)
        kinds = c.kernels(lambda: go(c.base.clone()))
        assert ("mfma_shrink" in kinds) and (product or "mfma_expand" in kinds)  # the lists with tiles
        for layer in () if product else (0, 39):
            c.check(eager[layer], layer, c.base[layer])
    finally:
        c.pool.close()


@pytest.mark.parametrize("call", ["list", "base product"])
def test_captured_behind_uploads_of_another_stream(call):
    """A plan and a slot's weights that another stream still has before it when the call is captured: they are there for the replays, which nothing orders behind that stream."""
    product = call == "base product"
    c = Case([200, 90, 77], 2048, 1024, 8) if product else Case(LENS[0], 512, 1024, 40)
    try:
        B, space = c.B, torch.empty(c.T * 1024, dtype=torch.float32, device="cuda")
        other, mine, graph = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.CUDAGraph()

        def go(y, stream):
            if product:
                B.check(B.lora_linear_plan(c.pool.handle, c.plan, 0, 0, c.x[0].data_ptr(), c.wt.data_ptr(), y.data_ptr(), 2.0, stream, space.data_ptr(), space.numel() * 4))
            else:
                c.apply_list(y, stream)

        y, busy = c.base.clone(), torch.randn(4096, 4096, device="cuda")
        c.pool.plan_destroy(c.plan)
        B.check(B.lora_cache_release_slot(c.pool.handle, 0))
        c.A[0], c.Bm[0] = -c.A[0], c.Bm[0] * 2  # slot 0 is filled anew
        a, b = c.A[0].cpu().pin_memory(), c.Bm[0].cpu().pin_memory()
        parts = B.make_fill_parts([(layer, 0, a.data_ptr(), b.data_ptr()) for layer in range(c.n_layers)])
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for _ in range(40):
                busy @ busy
            B.check(B.lora_cache_fill_slot_parts(c.pool.handle, 0, 99, int(c.rank_of[0]), 0.5, parts, other.cuda_stream))
            c.plan = c.pool.plan(c.T, c.off, c.slot, c.rank_of[c.slot])
            assert not other.query()
        with torch.cuda.stream(mine):
            graph.capture_begin(capture_error_mode="thread_local")
            go(y, mine.cuda_stream)
            graph.capture_end()
            graph.replay()
        torch.cuda.synchronize()
        eager = c.base.clone()
        go(eager, c.stream)
        c.pool.check_fault()
        assert torch.equal(y, eager)
        for layer in () if product else range(c.n_layers):
            c.check(y[layer], layer, c.base[layer])
    finally:
        c.pool.close()


@pytest.mark.parametrize("first", ["list", "base product"])
def test_calls_on_a_second_stream(first):
    """The lists' upload is behind work of the stream that made the plan; a call on another stream waits for it."""
    c = Case([200, 90, 77], 2048, 1024, 8)
    try:
        B, space = c.B, torch.empty(c.T * 1024, dtype=torch.float32, device="cuda")

        def product(y, stream):
            B.check(B.lora_linear_plan(c.pool.handle, c.plan, 0, 0, c.x[0].data_ptr(), c.wt.data_ptr(), y.data_ptr(), 2.0, stream, space.data_ptr(), space.numel() * 4))

        go = (lambda y, s: c.apply_list(y, s)) if first == "list" else product
        want = c.base.clone()
        go(want, c.stream)
        kinds = c.kernels(lambda: go(c.base.clone(), c.stream))
        assert "mfma_shrink" in kinds
        y, busy, done = c.base.clone(), Busy(), torch.cuda.Event()
        c.pool.plan_destroy(c.plan)
        other, mine = busy.one, busy.two  # (no apply has run on `other`: the lists do not wait for their first launch)
        torch.cuda.synchronize()
        busy.start()
        done.record(other)
        with torch.cuda.stream(other):
            c.plan = c.pool.plan(c.T, c.off, c.slot, c.rank_of[c.slot])
        go(y, mine.cuda_stream)
        assert not done.query()
        mine.synchronize()
        assert done.query()
        torch.cuda.synchronize()
        c.pool.check_fault()
        assert torch.equal(y, want)
    finally:
        c.pool.close()


@pytest.mark.parametrize("short", [1, 8, 30])
def test_a_pool_of_fewer_bytes(short, monkeypatch):
    """A byte short, and 8 and 30 of 44 sets (1 KB a token each): lists run in smaller batches, with tiles where a batch still gains by them (14 entries do not)."""
    from paper_2411_17741_amd import binding as B0

    required = B0.lora_cache_bytes_required
    monkeypatch.setattr(B0, "lora_cache_bytes_required", lambda cfg: required(cfg) - (1 if short == 1 else short * 1024 * cfg.max_tokens))
    c = Case(LENS[0], 512, 1024, 40)
    try:
        y = c.base.clone()
        c.B.lora_cache_set_timing(c.pool.handle, 1)
        c.apply_list(y)
        torch.cuda.synchronize()
        c.pool.check_fault()
        rc, t = c.B.lora_cache_read_timing(c.pool.handle)
        expands, gemv = t["mfma_expand"][1], t["gemv_fused"][1]
        assert rc == c.B.LORA_OK and (expands, gemv > 1) == {1: (1, False), 8: (1, True), 30: (0, True)}[short], t
        for layer in range(c.n_layers):
            c.check(y[layer], layer, c.base[layer])
    finally:
        c.pool.close()
