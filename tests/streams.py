"""Streams for tests in which one has work before it while another goes on."""
import torch


class Busy:
    """A stream `one` with a chain of products for it, and a stream `two` that does not share its hardware queue (a process has a few of them, streams take turns in them)."""

    def __init__(self):
        self.a = torch.randn(4096, 4096, device="cuda")
        self.one, word = torch.cuda.Stream(), torch.zeros(1, device="cuda")
        torch.cuda.synchronize()
        for _ in range(8):
            self.two = torch.cuda.Stream()
            self.start(10)
            early = torch.cuda.Event()
            early.record(self.one)
            self.start(10)
            with torch.cuda.stream(self.two):
                word.add_(1)
            self.two.synchronize()
            free = not early.query()  # (a shared queue: behind all of them)
            torch.cuda.synchronize()
            if free:
                return
        raise RuntimeError("no stream beside a busy one")

    def start(self, n=60):  # about a millisecond each
        with torch.cuda.stream(self.one):
            for _ in range(n):
                self.a @ self.a
