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
