"""The scratch of extract when it is out of order, as calls leave it that share it and overlap: the state is written from the host, and
the next call must say so (SRS_FLAG_TIMEOUT) and the one after srs_status be right again.  Every launch below ends by itself: no
tile is waited for that no workgroup takes."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
T = 8192


class Scratch:
    """Device words of a context, by the first members of srs_ctx (csrc/srs.hip): device, static scratch, the arrays
    of status words and of ticket counters (where, how many, where and how many at first), flag word (the epoch 32 words behind it, the count of claimed buckets 16 behind that)."""

    def __init__(self, ctx):
        at = lambda k: C.c_uint64.from_address(ctx._h.value + k).value  # noqa: E731
        self.static, self.status, self.status_cap, self.tickets, self.flags = at(8), at(16), at(24), at(48), at(80)
        self.epoch, self.claimed = self.flags + 128, self.flags + 192
        self.static_tickets = self.static + (8 << 20)
        self.static_epoch = self.static_tickets + (4 << 18)
        self.hip = C.CDLL(next(x.split()[-1] for x in open("/proc/self/maps") if "libamdhip64" in x))

    def read(self, address, words):
        torch.cuda.synchronize()
        a = np.zeros(words, np.uint32)
        assert self.hip.hipMemcpy(a.ctypes.data_as(C.c_void_p), C.c_void_p(address), C.c_size_t(a.nbytes), C.c_int(2)) == 0
        return a

    def write(self, address, value):
        torch.cuda.synchronize()
        a = np.array([value], np.uint32)
        assert self.hip.hipMemcpy(C.c_void_p(address), a.ctypes.data_as(C.c_void_p), C.c_size_t(4), C.c_int(1)) == 0
        torch.cuda.synchronize()


class Call:
    """Extract of `tiles` tiles in buckets of `per`, as one tensor, from a bitmap, or on the static scratch."""

    def __init__(self, ctx, kind, tiles, per, seed=1):
        from paper_2605_07330_amd import srs
        rng = np.random.default_rng(seed)
        n = tiles * T
        self.ctx, self.kind, self.be = ctx, kind, per * T
        self.old = rng.integers(0, 1 << 16, n).astype(np.uint16)
        self.new = (self.old ^ (rng.random(n) < 0.02)).astype(np.uint16)
        self.want = oracle.extract(self.old.copy(), self.new, self.be, self.be)[:3]
        self.t = torch.empty(n, dtype=torch.int16, device=DEV)
        self.u = torch.from_numpy(self.new.view(np.int16)).to(DEV)
        self.I, self.V, self.counts = srs.alloc_payload(-(-tiles // per), self.be, DEV)
        if kind == "marked":
            bits = np.packbits(self.old != self.new, bitorder="little").view(np.int32)
            self.bits = torch.from_numpy(bits.copy()).to(DEV)
            self.plan = ctx.plan([n], self.be)

    def run(self):
        self.t.copy_(torch.from_numpy(self.old.view(np.int16)))
        self.counts.fill_(-1)
        self.launch()

    def launch(self):
        a = (self.I, self.V, self.counts, self.be)
        if self.kind == "marked":
            self.ctx.extract_marked_multi(self.plan, [self.u], self.bits, *a)
        else:
            (self.ctx.extract_noalloc if self.kind == "static" else self.ctx.extract)(self.t, self.u, self.be, *a)

    def check(self):
        wI, wV, wc = self.want
        assert np.array_equal(self.counts.cpu().numpy().view(np.uint32), wc)
        I, V = self.I.cpu().numpy().reshape(len(wc), -1), self.V.cpu().numpy().view(np.uint16).reshape(len(wc), -1)
        for b, c in enumerate(wc):
            at = b * self.be if self.kind == "marked" else 0
            assert np.array_equal(I[b, :c] + at, wI[b, :c]) and np.array_equal(V[b, :c], wV[b, :c])


@pytest.fixture
def ctx():
    from paper_2605_07330_amd import srs
    c = srs.Context(0)
    c.set_option(srs.OPT_TILE_ELEMS, T)
    yield c
    c.close()


@pytest.mark.parametrize("kind", ["one", "marked"])
@pytest.mark.parametrize("fault", ["ticket", "epoch"])
def test_scratch_out_of_order_is_reported(ctx, kind, fault):
    from paper_2605_07330_amd import srs
    s, call = Scratch(ctx), Call(ctx, kind, 3, 3)
    call.run()
    assert ctx.status() == 0
    call.check()
    if fault == "ticket":                    # beyond this bucket's last: one of its three tiles is never served
        s.write(s.tickets, 5)
    else:                                    # not raised by the last launch, whose status words then look like this one's
        s.write(s.epoch, int(s.read(s.epoch, 1)[0]) - 1)
    call.run()
    assert ctx.status() == srs.FLAG_TIMEOUT
    call.run()
    assert ctx.status() == 0
    call.check()


def test_only_a_call_on_the_static_scratch_rewinds_it(ctx):
    """It belongs to every context of the GPU, whose calls on it need not be ordered with this one's look at its flags."""
    from paper_2605_07330_amd import srs
    s, own, static = Scratch(ctx), Call(ctx, "one", 3, 3), Call(ctx, "static", 5, 5)
    static.run()
    assert ctx.status() == 0
    before = int(s.read(s.static_epoch, 1)[0])
    assert before > 0
    s.write(s.tickets, 5)
    own.run()
    assert ctx.status() == srs.FLAG_TIMEOUT
    assert int(s.read(s.static_epoch, 1)[0]) == before and s.read(s.static, 8).any()
    s.write(s.static_tickets, 7)
    static.run()
    assert ctx.status() == srs.FLAG_TIMEOUT
    assert not s.read(s.static, 8).any() and int(s.read(s.static_tickets, 1)[0]) == 0
    static.run()
    own.run()
    assert ctx.status() == 0
    static.check()
    own.check()


def test_no_word_outlives_the_epochs(ctx):
    """A word that one layout's launch wrote is overwritten by launches that have a tile of a chain there, and wiped elsewhere, also where a
    tile is alone in its bucket: none can meet its own epoch again when that comes round."""
    s, long, short = Scratch(ctx), Call(ctx, "one", 40, 40), Call(ctx, "one", 5, 2)      # the short one: buckets of 2, 2 and 1 tiles
    long.run()
    assert ctx.status() == 0
    epoch = int(s.read(s.epoch, 1)[0]) - 1
    short.run()
    assert ctx.status() == 0
    words = s.read(s.status, 80).reshape(-1, 2)[:, 1]
    assert (words[5:39] != 0).all() and (words[[1, 3]] == 0).all() and (words[[0, 2]] >> 2 == epoch + 1).all(), words
    for _ in range(max(s.status_cap // 64, 1 << 14) + 1):
        short.launch()
    short.run()
    assert ctx.status() == 0
    short.check()
    words = s.read(s.status, 2 * s.status_cap).reshape(-1, 2)[:, 1]
    assert (words[5:] == 0).all() and (words[[1, 3, 4]] == 0).all()
    long.run()
    assert ctx.status() == 0
    long.check()
