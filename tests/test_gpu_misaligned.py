"""Extract on tiles that start anywhere against the 16-byte vectors (snapshot and new weights each by their own offset) and end
anywhere, against the oracle, tolerance 0: the incomplete vectors in front and behind, tiles of one or two vectors, the
grid that ends one element before, at or after a whole tile, lines that cross the rows of a wave; both element widths,
the fused cast, and every way to refresh the snapshot.  What lies before and after the tensors stays as it was."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
PAD = 96
SIZES = [1, 3, 7, 8, 9, 15, 17, 31, 33, 2047, 4095, 4096, 4097, 8191, 8193, 12303, 32760, 32767, 32768, 32769, 32775, 40001]


def device_copy(a, pad):
    """The array on the GPU, `pad` elements into a filled buffer: (buffer, the view)."""
    buf = np.full(a.size + pad + PAD, 0x77, a.dtype)
    buf[pad:pad + a.size] = a
    t = torch.from_numpy(buf.view(np.int16) if a.dtype == np.uint16 else buf).to(DEV)
    return t, t[pad:pad + a.size], buf


def host(t, dt):
    return t.cpu().numpy().view(dt)


@pytest.mark.parametrize("tile", [32768, 8192])
@pytest.mark.parametrize("mode,kind", [(mode, kind) for mode in ("lines", "elements", "rotate", "second") for kind in ("bf16", "u8", "cast")
                                       if kind != "cast" or mode in ("lines", "elements")])      # the cast has no snapshot option
@pytest.mark.parametrize("oo,no", [(0, 0), (1, 1), (8, 0), (3, 5), (7, 2), (24, 24), (61, 60)])
def test_extract_any_alignment(oo, no, mode, tile, kind):
    from paper_2605_07330_amd import srs
    print(f"case old+{oo} new+{no} {mode} tile={tile} {kind}", flush=True)
    dt = np.uint8 if kind == "u8" else np.uint16
    rng = np.random.default_rng(100 * oo + no)
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_TILE_ELEMS, tile)
        ctx.set_option(srs.OPT_REFRESH_GROUP, 0 if mode == "elements" else 8)
        ctx.set_option(srs.OPT_SNAPSHOT, {"rotate": 1, "second": 2}.get(mode, 0))
        for n in SIZES:
            for density in (0.02, 0.7):
                be = n if n < 9000 else n // 2 + 3
                cap = be
                old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
                if kind == "cast":
                    m = (rng.standard_normal(n) * 0.02).astype(np.float32)
                    old = np.where(rng.random(n) < density, old, oracle.round_bf16(m)).astype(np.uint16)
                    new = m
                else:
                    new = np.where(rng.random(n) < density, rng.integers(0, 1 << (8 * dt().itemsize), n), old).astype(dt)
                    new[0], new[-1] = ~old[0], ~old[-1]
                want_old = old.copy()
                fn = {"bf16": oracle.extract, "u8": oracle.extract_u8, "cast": oracle.extract_cast}[kind]
                wI, wV, wc = fn(want_old, new, be, cap)[:3]
                if mode == "rotate":
                    want_old = old
                tb, t, buf = device_copy(old, oo)
                _, u, _ = device_copy(new, no)
                alloc = srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload
                I, V, counts = alloc(len(wc), cap, DEV)
                run = {"bf16": ctx.extract, "u8": ctx.extract_u8, "cast": ctx.extract_cast}[kind]
                run(t, u, be, I, V, counts, cap)
                assert ctx.status() == 0
                gc = counts.cpu().numpy().view(np.uint32)[:len(wc)]
                assert np.array_equal(gc, wc), n
                gI, gV = I.cpu().numpy().reshape(len(wc), cap), host(V, dt).reshape(len(wc), cap)
                for b, c in enumerate(wc):
                    assert np.array_equal(gI[b, :c], wI[b, :c]) and np.array_equal(gV[b, :c], wV[b, :c]), (n, b)
                buf[oo:oo + n] = want_old
                assert np.array_equal(host(tb, dt), buf), n
    finally:
        ctx.close()


@pytest.mark.parametrize("cast", [False, True])
@pytest.mark.parametrize("tile", [32768, 4096])
@pytest.mark.parametrize("oo,no", [(0, 0), (1, 3), (7, 2), (61, 60)])
def test_mark_any_alignment(oo, no, tile, cast):
    """Tensors end to end in one buffer, so that each starts at its own offset, in tiles that the buckets cut anywhere."""
    from paper_2605_07330_amd import srs
    print(f"case mark old+{oo} new+{no} tile={tile} cast={cast}", flush=True)
    total, be = sum(SIZES), 20011
    for density in (0.02, 0.7):
        rng = np.random.default_rng(100 * oo + no)
        old = rng.integers(0, 1 << 16, total).astype(np.uint16)
        change = rng.random(total) < density
        change[[0, -1]] = True
        if cast:
            new = (rng.standard_normal(total) * 0.02).astype(np.float32)
            old = np.where(change, old, oracle.round_bf16(new)).astype(np.uint16)
        else:
            new = np.where(change, ~old, old).astype(np.uint16)
        cuts = np.cumsum([0] + SIZES)
        views = lambda t: [t[a:b] for a, b in zip(cuts[:-1], cuts[1:])]  # noqa: E731
        want, bits = old.copy(), np.zeros(oracle.bitmap_words(total), np.uint32)
        (oracle.cast_mark_multi if cast else oracle.mark_multi)(views(want), views(new), SIZES, bits)
        tb, t, buf = device_copy(old, oo)
        _, u, _ = device_copy(new, no)
        ctx = srs.Context(0)
        try:
            ctx.set_option(srs.OPT_TILE_ELEMS, tile)
            plan = ctx.plan(SIZES, be)
            guard = 5                                      # words on both sides of the bitmap stay clear
            words = torch.zeros(bits.size + 2 * guard, dtype=torch.int32, device=DEV)
            bitmap = words[guard:guard + bits.size]
            (ctx.cast_mark_multi if cast else ctx.mark_multi)(plan, views(t), views(u), bitmap)
            assert ctx.status() == 0
            assert np.array_equal(host(bitmap, np.uint32), bits)
            assert (words[:guard] == 0).all() and (words[guard + bits.size:] == 0).all()
            buf[oo:oo + total] = want
            assert np.array_equal(host(tb, np.uint16), buf)
        finally:
            ctx.close()


@pytest.mark.parametrize("oo,no", [(0, 0), (1, 3), (7, 2), (61, 60)])
def test_dense_copy_any_alignment(oo, no):
    """Every bucket packed whole and unpacked into other weights; slots of an odd size, so that they too start anywhere."""
    from paper_2605_07330_amd import srs
    print(f"case dense new+{no} weights+{oo}", flush=True)
    total, be = sum(SIZES), 20011
    rng = np.random.default_rng(100 * oo + no)
    new = rng.integers(0, 1 << 16, total).astype(np.uint16)
    cuts = np.cumsum([0] + SIZES)
    views = lambda t: [t[a:b] for a, b in zip(cuts[:-1], cuts[1:])]  # noqa: E731
    ctx = srs.Context(0)
    try:
        plan = ctx.plan(SIZES, be)
        nb = plan.nbuckets
        _, u, _ = device_copy(new, no)
        tb, t, buf = device_copy(np.zeros(total, np.uint16), oo)
        order = rng.permutation(nb).astype(np.int32)
        bucket_of = torch.from_numpy(order).to(DEV)
        n_dense = torch.full((1,), nb, dtype=torch.int32, device=DEV)
        dense = torch.zeros(nb * be + PAD, dtype=torch.int16, device=DEV)
        ctx.pack_dense_multi(plan, views(u), views(u), bucket_of, n_dense, nb, dense)
        want = np.zeros(nb * be + PAD, np.uint16)
        for s, b in enumerate(order):
            run = new[b * be:(b + 1) * be]
            want[s * be:s * be + run.size] = run
        assert np.array_equal(host(dense, np.uint16), want)
        ctx.unpack_dense_multi(plan, views(t), bucket_of, n_dense, nb, dense)
        assert ctx.status() == 0
        buf[oo:oo + total] = new
        assert np.array_equal(host(tb, np.uint16), buf)
    finally:
        ctx.close()
