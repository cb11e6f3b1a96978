"""Tiles that do not fill their workgroup: lengths around every four vectors of a wave (what an incomplete tile loads or leaves out
together), around the waves' shares, a vector and a whole tile, at every alignment, against the oracle, tolerance 0."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def lengths(tile, ve):
    """Tensor lengths of a list; each is a tile of its own (or two)."""
    row = 64 * ve
    at = {1, 2, ve, 2 * ve, row, tile // 4, tile // 2, tile - row, tile, tile + row}
    at |= {4 * row * k for k in range(1, tile // (4 * row) + 1)}
    return sorted({max(1, a + d) for a in at for d in (-ve - 1, -1, 0, 1, ve + 3)})


@pytest.mark.parametrize("mode", ["lines", "elements", "rotate"])
@pytest.mark.parametrize("kind,tile", [("bf16", 32768), ("bf16", 8192), ("bf16", 4096), ("u8", 32768), ("u8", 8192), ("cast", 32768), ("cast", 16384), ("cast", 4096)])
def test_lengths_around_the_loads(kind, tile, mode):
    from paper_2605_07330_amd import srs
    if kind == "cast" and mode == "rotate":
        pytest.skip("the cast has no snapshot option")
    print(f"case {kind} tile={tile} {mode}", flush=True)
    dt = np.uint8 if kind == "u8" else np.uint16
    rng = np.random.default_rng(tile)
    numel = [int(x) for x in rng.permutation(lengths(tile, 16 // dt().itemsize))]
    n, be = sum(numel), 5 * tile + 13                        # a bucket holds several tensors and cuts some
    mask = rng.random(n) < 0.02
    mask[np.cumsum([0, *numel[:-1]])] = True                 # the first and the last element of each tensor
    mask[np.cumsum(numel) - 1] = True
    if kind == "cast":
        new = (rng.standard_normal(n) * 0.02).astype(np.float32)
        old = (oracle.round_bf16(new) ^ mask.astype(np.uint16)).astype(np.uint16)
    else:
        old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
        new = (old ^ mask.astype(dt)).astype(dt)
    split = lambda a: [np.ascontiguousarray(x) for x in np.split(a, np.cumsum(numel)[:-1])]  # noqa: E731
    after = [x.copy() for x in split(old)]
    name = {"bf16": "extract_multi", "u8": "extract_multi_u8", "cast": "extract_cast_multi"}[kind]
    wI, wV, wc = getattr(oracle, name)(after, split(new), numel, be, be)[:3]
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        ctx.set_option(srs.OPT_REFRESH_GROUP, 0 if mode == "elements" else 8)
        ctx.set_option(srs.OPT_SNAPSHOT, 1 if mode == "rotate" else 0)
        plan = ctx.plan(numel, be)
        as_torch = lambda a: torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).to(DEV)  # noqa: E731
        t, u = as_torch(old.copy()), as_torch(new)           # end to end: every alignment
        I, V, counts = (srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload)(plan.nbuckets, be, DEV)
        getattr(ctx, name)(plan, list(torch.split(t, numel)), list(torch.split(u, numel)), I, V, counts, be)
        assert ctx.status() == 0
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), wc)
        gI, gV = I.cpu().numpy().reshape(len(wc), be), V.cpu().numpy().view(dt).reshape(len(wc), be)
        for b, c in enumerate(wc):
            assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), b
        assert np.array_equal(t.cpu().numpy().view(dt), old if mode == "rotate" else np.concatenate(after))
        plan.close()
    finally:
        ctx.close()


@pytest.mark.parametrize("mode", ["lines", "rotate"])
@pytest.mark.parametrize("kind,tile", [("bf16", 32768), ("cast", 32768), ("u8", 32768), ("bf16", 8192)])
@pytest.mark.parametrize("per", [1, 3, 40])
def test_pairs_around_what_one_wave_writes_out(kind, tile, mode, per):
    """Tiles with as many pairs as one wave still writes out, one fewer and one more, and full rounds, in chains and alone in their
    buckets; a capacity that cuts some off."""
    from paper_2605_07330_amd import srs
    if kind == "cast" and mode == "rotate":
        pytest.skip("the cast has no snapshot option")
    print(f"case {kind} tile={tile} {mode} per={per}", flush=True)
    dt = np.uint8 if kind == "u8" else np.uint16
    rng = np.random.default_rng(per)
    n, be = 40 * tile, per * tile
    mask = np.zeros(n, bool)
    for k in range(40):
        mask[k * tile + rng.permutation(tile)[:int(rng.choice([0, 1, 64, 1023, 1024, 1025, 2047, 2048]))]] = True
    if kind == "cast":
        new = (rng.standard_normal(n) * 0.02).astype(np.float32)
        old = (oracle.round_bf16(new) ^ mask.astype(np.uint16)).astype(np.uint16)
    else:
        old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
        new = (old ^ mask.astype(dt)).astype(dt)
    cap, after = per * 1200, old.copy()
    wI, wV, wc = {"bf16": oracle.extract, "u8": oracle.extract_u8, "cast": oracle.extract_cast}[kind](after, new, be, cap)[:3]
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        ctx.set_option(srs.OPT_SNAPSHOT, 1 if mode == "rotate" else 0)
        as_torch = lambda a: torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).to(DEV)  # noqa: E731
        t, u = as_torch(old.copy()), as_torch(new)
        I, V, counts = (srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload)(len(wc), cap, DEV)
        {"bf16": ctx.extract, "u8": ctx.extract_u8, "cast": ctx.extract_cast}[kind](t, u, be, I, V, counts, cap)
        assert ctx.status() == (srs.FLAG_OVERFLOW if (np.asarray(wc) > cap).any() else 0)
        assert np.array_equal(counts.cpu().numpy().view(np.uint32)[:len(wc)], wc)
        gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().view(dt).reshape(len(wc), cap)
        for b, c in enumerate(np.minimum(wc, cap)):
            assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), b
        assert np.array_equal(t.cpu().numpy().view(dt), old if mode == "rotate" else after)
    finally:
        ctx.close()


@pytest.mark.parametrize("mode", ["lines", "elements", "rotate", "second"])
@pytest.mark.parametrize("form", ["whole", "most", "nine", "eight", "shifted", "one_shifted", "chains", "fewer_chains"])
def test_lists_of_whole_tiles(form, mode):
    """Lists on both sides of the share of whole aligned tiles from which another kernel takes them, one with a few tensors off the
    16-byte boundaries, and the plan called again with other pointers."""
    from paper_2605_07330_amd import srs
    T = 32768
    numel = {"whole": [3 * T] * 12, "most": [19 * T + 40, 8, 17 * T + 8, T], "nine": [9 * T + 24] * 4, "eight": [8 * T + 24] * 4, "shifted": [6 * T] * 5,
             "one_shifted": [2 * T] * 6 + [7, 13 * T + 24] + [2 * T] * 3, "chains": [64 * T] * 4, "fewer_chains": [64 * T] * 3 + [62 * T]}[form]
    print(f"case {form} {mode}", flush=True)
    rng = np.random.default_rng(len(form))
    n, be = sum(numel), 2 * T if form.endswith("chains") else 8 * T + 512      # 128 and 127 buckets of two tiles
    pad = [0 if form != "shifted" else 1 for _ in numel]     # elements in front of each tensor
    if form == "one_shifted":
        pad[3] = 3
    as_torch = lambda a: torch.from_numpy(a.view(np.int16)).to(DEV)  # noqa: E731
    split = lambda a: [np.ascontiguousarray(x) for x in np.split(a, np.cumsum(numel)[:-1])]  # noqa: E731
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_REFRESH_GROUP, 0 if mode == "elements" else 8)
        ctx.set_option(srs.OPT_SNAPSHOT, {"rotate": 1, "second": 2}.get(mode, 0))
        plan = ctx.plan(numel, be)
        for again in range(3):
            if again == 1:                                  # the same list, off or on the boundaries
                pad = [1 - min(p, 1) for p in pad]
            old = rng.integers(0, 1 << 16, n).astype(np.uint16)
            new = (old ^ (rng.random(n) < (0.004, 0.04, 0.2)[again])).astype(np.uint16)
            after = [x.copy() for x in split(old)]
            wI, wV, wc = oracle.extract_multi(after, split(new), numel, be, be)[:3]
            put = lambda a: [torch.empty(len(x) + p, dtype=torch.int16, device=DEV)[p:].copy_(as_torch(x)) for x, p in zip(split(a), pad)]  # noqa: E731
            t, u = put(old), put(new)
            I, V, counts = srs.alloc_payload(plan.nbuckets, be, DEV)
            ctx.extract_multi(plan, t, u, I, V, counts, be)
            assert ctx.status() == 0
            assert np.array_equal(counts.cpu().numpy().view(np.uint32), wc)
            gI, gV = I.cpu().numpy().reshape(len(wc), be), V.cpu().numpy().view(np.uint16).reshape(len(wc), be)
            for b, c in enumerate(wc):
                assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), b
            got = np.concatenate([x.cpu().numpy().view(np.uint16) for x in t])
            assert np.array_equal(got, old if mode == "rotate" else np.concatenate(after))
        plan.close()
    finally:
        ctx.close()


@pytest.mark.parametrize("tile", [32768, 4096])
@pytest.mark.parametrize("per", [1, 2])
def test_marked_pairs_around_one_each(tile, per):
    """The payload of a bitmap where tiles hold about as many pairs as there are threads, alone in their buckets or two in one, whole and
    short ones; a capacity that cuts some off."""
    from paper_2605_07330_amd import srs
    print(f"case tile={tile} per={per}", flush=True)
    rng = np.random.default_rng(tile + per)
    numel = [30 * tile, 7, 3 * tile + 300, 5]
    n, be = sum(numel), per * tile
    mask = np.zeros(n, bool)
    for lo in range(0, n, tile):
        hi = min(n, lo + tile)
        mask[lo + rng.permutation(hi - lo)[:int(rng.choice([0, 1, 64, 200, 255, 256, 257, 300]))]] = True
    new = rng.integers(0, 1 << 16, n).astype(np.uint16)
    split = lambda a: [np.ascontiguousarray(x) for x in np.split(a, np.cumsum(numel)[:-1])]  # noqa: E731
    bits = np.zeros(oracle.bitmap_words(n), np.uint32)
    oracle.mark_multi(split(new ^ mask), split(new), numel, bits)
    cap = 250 * per
    wI, wV, wc = oracle.extract_marked_multi(split(new), numel, be, bits, cap)[:3]
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        plan = ctx.plan(numel, be)
        I, V, counts = srs.alloc_payload(plan.nbuckets, cap, DEV)
        flat = torch.from_numpy(new.view(np.int16)).to(DEV)
        ctx.extract_marked_multi(plan, list(torch.split(flat, numel)), torch.from_numpy(bits.view(np.int32)).to(DEV), I, V, counts, cap)
        assert ctx.status() == srs.FLAG_OVERFLOW and (wc > cap).any()
        assert np.array_equal(counts.cpu().numpy().view(np.uint32), wc)
        gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().view(np.uint16).reshape(len(wc), cap)
        for b, c in enumerate(np.minimum(wc, cap)):
            assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), b
            assert (gI[b, c:] == -1).all()
        plan.close()
    finally:
        ctx.close()
