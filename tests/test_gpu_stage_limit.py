"""Tiles whose pairs just fit the one round that a single wave writes out, and tiles that need more, side by side on one chain:
counts of changed elements per tile at the edges of a wave and of the stage (2048 pairs), against the oracle, tolerance 0."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
COUNTS = [0, 1, 63, 64, 65, 2047, 2048, 2049, 4095]


@pytest.mark.parametrize("mode", ["lines", "elements", "rotate"])
@pytest.mark.parametrize("kind,tile", [("bf16", 32768), ("bf16", 16384), ("bf16", 4096), ("u8", 32768), ("u8", 8192), ("cast", 32768), ("cast", 4096)])
def test_pairs_of_a_tile_around_the_stage(kind, tile, mode):
    from paper_2605_07330_amd import srs
    if kind == "cast" and mode == "rotate":
        pytest.skip("the cast has no snapshot option")
    print(f"case {kind} tile={tile} {mode}", flush=True)
    dt = np.uint8 if kind == "u8" else np.uint16
    rng = np.random.default_rng(tile)
    ntiles = 90
    n = (ntiles - 1) * tile + tile // 2 + 5
    be = 70 * tile                                              # a bucket of 70 tiles, a shorter one behind it
    mask = np.zeros(n, bool)
    for k in range(ntiles):
        lo, hi = k * tile, min(n, (k + 1) * tile)
        c = min(int(rng.choice(COUNTS)), hi - lo)
        mask[lo + rng.permutation(hi - lo)[:c]] = True
    if kind == "cast":
        new = (rng.standard_normal(n) * 0.02).astype(np.float32)
        old = (oracle.round_bf16(new) ^ mask.astype(np.uint16)).astype(np.uint16)
    else:
        old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
        new = (old ^ mask.astype(dt)).astype(dt)
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        ctx.set_option(srs.OPT_REFRESH_GROUP, 0 if mode == "elements" else 8)
        ctx.set_option(srs.OPT_SNAPSHOT, 1 if mode == "rotate" else 0)
        want_old = old.copy()
        fn = {"bf16": oracle.extract, "u8": oracle.extract_u8, "cast": oracle.extract_cast}[kind]
        cap = 70 * 4096
        wI, wV, wc = fn(want_old, new, be, cap)[:3]
        as_torch = lambda a: torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).to(DEV)  # noqa: E731
        t, u = as_torch(old.copy()), as_torch(new)
        I, V, counts = (srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload)(len(wc), cap, DEV)
        {"bf16": ctx.extract, "u8": ctx.extract_u8, "cast": ctx.extract_cast}[kind](t, u, be, I, V, counts, cap)
        assert ctx.status() == 0
        assert np.array_equal(counts.cpu().numpy().view(np.uint32)[:len(wc)], wc)
        gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().view(dt).reshape(len(wc), cap)
        for b, c in enumerate(wc):
            assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), b
        assert np.array_equal(t.cpu().numpy().view(dt), old if mode == "rotate" else want_old)
    finally:
        ctx.close()


@pytest.mark.parametrize("tile", [32768, 16384, 8192, 4096])
@pytest.mark.parametrize("lead", [0, 5, 31, 32])
def test_marked_pairs_of_a_tile_around_the_stage(tile, lead):
    """The same for the payload of a bitmap, the tiles starting `lead` bits into a word of it; the last slice ends with the bitmap."""
    from paper_2605_07330_amd import srs
    print(f"case marked tile={tile} lead={lead}", flush=True)
    rng = np.random.default_rng(tile + lead)
    numel = ([lead] if lead else []) + [40 * tile + 96, 3 * tile // 2 + 7]
    n, be = sum(numel), 25 * tile
    mask = np.zeros(n, bool)
    for lo in range(lead, n, tile):
        hi = min(n, lo + tile)
        mask[lo + rng.permutation(hi - lo)[:min(int(rng.choice(COUNTS)), hi - lo)]] = True
    mask[-1] = True
    new = rng.integers(0, 1 << 16, n).astype(np.uint16)
    split = lambda a: [np.ascontiguousarray(x) for x in np.split(a, np.cumsum(numel)[:-1])]  # noqa: E731
    bits = np.zeros(oracle.bitmap_words(n), np.uint32)
    oracle.mark_multi(split(new ^ mask), split(new), numel, bits)
    cap = 3000 * 25
    want = oracle.extract_marked_multi(split(new), numel, be, bits, cap)[:3]
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        plan = ctx.plan(numel, be)
        flat = torch.from_numpy(new.view(np.int16)).to(DEV)
        I, V, counts = srs.alloc_payload(plan.nbuckets, cap, DEV)
        ctx.extract_marked_multi(plan, list(torch.split(flat, numel)), torch.from_numpy(bits.view(np.int32)).to(DEV), I, V, counts, cap)
        assert ctx.status() == 0
        wI, wV, wc = want
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), wc)
        gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().view(np.uint16).reshape(len(wc), cap)
        for b, c in enumerate(wc):
            assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), b
        plan.close()
    finally:
        ctx.close()


def test_marked_gather_of_a_large_list():
    """More than 2^29 elements, whose gathers carry another cache hint: every value against the weights on the device."""
    from paper_2605_07330_amd import srs
    n, be = (1 << 29) + 12_345, 1 << 25
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    new = torch.randint(-32768, 32768, (n,), dtype=torch.int16, device=DEV, generator=g)
    bits = torch.zeros((n + 31) // 32, dtype=torch.int32, device=DEV)
    word = torch.randint(0, bits.numel() - 1, (bits.numel() // 4,), device=DEV, generator=g).unique()
    bits[word] = (1 << 17) | 5
    at = (word[:, None] * 32 + torch.tensor([0, 2, 17], device=DEV)).flatten()
    cap = be // 20
    ctx = srs.Context(0)
    try:
        plan = ctx.plan([n - 999, 999], be)
        I, V, counts = srs.alloc_payload(plan.nbuckets, cap, DEV)
        ctx.extract_marked_multi(plan, list(torch.split(new, [n - 999, 999])), bits, I, V, counts, cap)
        assert ctx.status() == 0
        assert torch.equal(counts.to(torch.int64), torch.bincount(at // be, minlength=plan.nbuckets))
        live = torch.arange(cap, device=DEV)[None, :] < counts[:, None]
        pos = (I.view(plan.nbuckets, cap) + torch.arange(plan.nbuckets, device=DEV)[:, None] * be)[live]
        assert torch.equal(pos, at) and torch.equal(V.view(plan.nbuckets, cap)[live], new[at])
        plan.close()
    finally:
        ctx.close()
