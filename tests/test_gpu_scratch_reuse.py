"""Tickets and tile status words are not cleared between launches: calls of every kind and of growing and shrinking size on one
context, with captured launches and launches that gave up between them, each against the oracle, tolerance 0."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = 4096


def dev(a):
    return torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).to(DEV)


class Call:
    """One extract of n elements in buckets of be on the context, run and checked."""

    def __init__(self, srs, ctx, kind, n, be, seed):
        rng = np.random.default_rng(seed)
        self.srs, self.ctx, self.kind, self.be, self.cap = srs, ctx, kind, be, be
        dt = np.uint8 if kind == "u8" else np.uint16
        self.old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
        self.new = (self.old ^ (rng.random(n) < 0.02)).astype(dt)
        self.dt, self.nb = dt, (n + be - 1) // be
        self.t, self.u = dev(self.old), dev(self.new)
        self.I, self.V, self.counts = (srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload)(self.nb, be, DEV)
        if kind in ("list", "marked"):
            cut = sorted({n // 3, n // 3 + n // 5})
            self.numel = list(np.diff([0, *cut, n]))
            self.plan = ctx.plan(self.numel, be)
            parts = lambda x: list(torch.split(x, self.numel))  # noqa: E731
            self.pairs = ctx.bind_pairs(self.plan, parts(self.t), parts(self.u))
            self.gather = ctx.plan(self.numel, be)    # a plan for each set of pointers: a captured upload would be replayed
            self.current = ctx.bind_weights(self.gather, parts(self.u))
            self.bitmap = torch.zeros(srs.bitmap_words(n), dtype=torch.int32, device=DEV)

    def launch(self):
        c, a = self.ctx, (self.I, self.V, self.counts, self.cap)
        if self.kind == "list":
            c.extract_multi(self.plan, None, None, *a, pairs=self.pairs)
        elif self.kind == "marked":
            c.mark_multi(self.plan, None, None, self.bitmap, pairs=self.pairs)
            c.extract_marked_multi(self.gather, None, self.bitmap, *a, tensors=self.current)
        else:
            {"one": c.extract, "static": c.extract_noalloc, "u8": c.extract_u8}[self.kind](self.t, self.u, self.be, *a)

    def reset(self):
        self.t.copy_(dev(self.old))
        self.counts.fill_(-1)
        if self.kind == "marked":
            self.bitmap.zero_()

    def check(self, where):
        fn = oracle.extract_u8 if self.kind == "u8" else oracle.extract
        wI, wV, wc = fn(self.old.copy(), self.new, self.be, self.cap)[:3]
        assert np.array_equal(self.counts.cpu().numpy().view(np.uint32)[:self.nb], wc), where
        gI, gV = self.I.cpu().numpy().reshape(self.nb, -1), self.V.cpu().numpy().view(self.dt).reshape(self.nb, -1)
        for b, c in enumerate(wc):
            at = b * self.be if self.kind in ("list", "marked") else 0           # positions in the bucket / in the tensor
            assert np.array_equal(gI[b, :c] + at, wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), (where, b)


SHAPES = [("one", 40 * T, 40 * T), ("u8", 9 * 8192 + 5, 3 * 8192), ("list", 70 * T + 11, 9 * T + 3), ("one", 3 * T, T), ("static", 33 * T + 1, 7 * T),
          ("marked", 50 * T + 100, 50 * T + 100), ("one", 300 * T + 7, 100 * T), ("static", 5 * T, 5 * T), ("list", 20 * T, 20 * T), ("one", T + 1, 2 * T)]


@pytest.mark.parametrize("tile", [8192, 0])
def test_calls_of_changing_size_share_the_scratch(tile):
    from paper_2605_07330_amd import srs
    ctx = srs.Context(0)
    try:
        if tile:
            ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        calls = [Call(srs, ctx, *s, seed=k) for k, s in enumerate(SHAPES)]
        for c in reversed(calls):                     # the largest status array and the pointer tables exist before the capture
            c.launch()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        captured = [calls[k] for k in (0, 2, 4, 5)]
        with torch.cuda.graph(g):
            for c in captured:
                c.launch()
        rng = np.random.default_rng(1)
        for step in range(60):
            if step % 7 == 3:
                for c in captured:
                    c.reset()
                g.replay()
                done = captured
            else:
                done = [calls[int(rng.integers(len(calls)))]]
                done[0].reset()
                done[0].launch()
            assert ctx.status() == 0
            for c in done:
                c.check(step)
    finally:
        ctx.close()


def test_a_launch_that_gave_up_leaves_the_scratch_usable():
    from paper_2605_07330_amd import srs
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, 8192)
        calls = [Call(srs, ctx, *s, seed=k) for k, s in enumerate(SHAPES)]
        for step in range(12):
            ctx.set_option(srs.OPT_SPIN_LIMIT, 1)
            big = calls[6 if step % 2 else 0]
            big.reset()
            big.launch()
            if step % 3:                              # with and without the look at the flags in between
                assert ctx.status() in (0, srs.FLAG_TIMEOUT)
            ctx.set_option(srs.OPT_SPIN_LIMIT, 1 << 24)
            for c in (calls[step % len(calls)], big):
                c.reset()
                c.launch()
                ctx.status()                          # the flag may still be the first launch's
                c.check(step)
    finally:
        ctx.close()
