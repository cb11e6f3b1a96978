"""Single tensors in a context that sets no tile size: around the sizes where the tile that the library picks changes, in one
bucket, several and one per tile, against the oracle, tolerance 0; buckets of one tile (no tickets, no status words) in
between calls that use both."""
import numpy as np
import pytest
import torch

import oracle
from util import assert_payload_equal, from_u16, payload_to_host, u16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CASES = [(n, be) for n in (1, 4096, 4097, 8192, 8193, 16384, 16385, 32768, 32769, 1 << 20, (1 << 20) + 1, (1 << 21) + 1,
                           1 << 22, (1 << 22) + 1, (1 << 23) + 1) for be in sorted({n, max(n // 4 - 1, 1), 9000, 16384, 40000})
         if be <= n]


@pytest.mark.parametrize("kind", ["bf16", "noalloc", "second", "cast", "u8"])
def test_single_tensor_default_tiles(kind):
    from paper_2605_07330_amd import srs
    ctx = srs.Context(0)
    try:
        if kind == "second":
            ctx.set_option(srs.OPT_SNAPSHOT, 2)
        for n, be in CASES:
            print(f"case {kind} n={n} be={be}", flush=True)
            rng = np.random.default_rng(n + be)
            dt = np.uint8 if kind == "u8" else np.uint16
            old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
            change = rng.random(n) < 0.02
            change[[0, -1]] = True
            if kind == "cast":
                new = (rng.standard_normal(n) * 0.02).astype(np.float32)
                old = np.where(change, old, oracle.round_bf16(new)).astype(np.uint16)
            else:
                new = np.where(change, ~old, old).astype(dt)
            cap = min(be, be // 20 + 64)                       # some of the small buckets overflow
            want_old = old.copy()
            fn = {"u8": oracle.extract_u8, "cast": oracle.extract_cast}.get(kind, oracle.extract)
            wI, wV, wc, overflow = fn(want_old, new, be, cap)
            t = torch.from_numpy(old.view(np.int16) if dt == np.uint16 else old).to(DEV)
            u = torch.from_numpy(new.view(np.int16) if new.dtype == np.uint16 else new).to(DEV)
            I, V, counts = (srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload)(len(wc), cap, DEV)
            run = {"noalloc": ctx.extract_noalloc, "u8": ctx.extract_u8, "cast": ctx.extract_cast}.get(kind, ctx.extract)
            run(t, u, be, I, V, counts, cap)
            assert ctx.status() == (srs.FLAG_OVERFLOW if overflow else 0)
            assert np.array_equal(counts.cpu().numpy().view(np.uint32)[:len(wc)], wc)
            gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().view(dt).reshape(len(wc), cap)
            live = np.arange(cap)[None, :] < np.minimum(wc, cap)[:, None]
            assert np.array_equal(gI[live], wI[live]) and np.array_equal(gV[live], wV[live])
            assert np.array_equal(t.cpu().numpy().view(dt), want_old)
    finally:
        ctx.close()


@pytest.mark.parametrize("be", [700, 4096, 32768])
def test_list_of_one_tile_buckets(be):
    """A list whose buckets hold one tile each, and one with more, in turn on the same context."""
    from paper_2605_07330_amd import srs
    rng = np.random.default_rng(be)
    ctx = srs.Context(0)
    try:
        for numel in ([be] * 70, [3 * be + 5, 9, be], [be] * 70):
            old = [rng.integers(0, 1 << 16, m).astype(np.uint16) for m in numel]
            new = [np.where(rng.random(o.size) < 0.1, ~o, o).astype(np.uint16) for o in old]
            bits = np.zeros(oracle.bitmap_words(sum(numel)), np.uint32)
            oracle.mark_multi(old, new, numel, bits)
            marked = oracle.extract_marked_multi(new, numel, be, bits)[:3]
            d_old, d_new = [from_u16(o, DEV) for o in old], [from_u16(w, DEV) for w in new]
            want = oracle.extract_multi(old, new, numel, be)[:3]
            plan = ctx.plan(numel, be)
            I, V, counts = srs.alloc_payload(plan.nbuckets, be, DEV)
            ctx.extract_multi(plan, d_old, d_new, I, V, counts, be)
            assert ctx.status() == 0
            assert_payload_equal(payload_to_host(I, V, counts), want, "list")
            assert all(np.array_equal(u16(a), b) for a, b in zip(d_old, new))
            bitmap = torch.from_numpy(bits.view(np.int32)).to(DEV)
            I, V, counts = srs.alloc_payload(plan.nbuckets, be, DEV)
            ctx.extract_marked_multi(plan, d_new, bitmap, I, V, counts, be)
            assert ctx.status() == 0
            assert_payload_equal(payload_to_host(I, V, counts), marked, "marked")
            plan.close()
    finally:
        ctx.close()
