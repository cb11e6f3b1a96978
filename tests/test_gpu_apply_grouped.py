"""Apply on payload slots that hold whole buckets, where a workgroup takes several chunks behind the first ones of a bucket:
counts around every chunk boundary, groups of two, four and eight chunks, buckets with few and with many segments next to each
other, an index out of range, and the second-pass snapshot refresh; against the same assignment by torch, tolerance 0."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 2048

# (buckets, bucket_elems): above 8192 slots, enough of them for each size of group; the last two on either side of 16 chunks
CASES = [(1, 17_000_001), (7, 9_000_000), (1500, 81_920), (1025, 30_721), (1025, 30_720)]


def make_payload(nb, be, n, width, multi, seed):
    """(I, V, counts, packed positions, values): counts at and around chunk boundaries, the first and the last bucket full."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    cpb = -(-be // CHUNK)
    counts = rng.integers(0, cpb + 1, nb) * CHUNK + rng.integers(-1, 2, nb)
    counts[[0, -1]] = be
    span = np.minimum(be, n - np.arange(nb) * be)
    counts = torch.from_numpy(np.clip(counts, 0, span)).to(DEV)
    span = torch.from_numpy(span).to(DEV)
    r = torch.arange(be, dtype=torch.int32, device=DEV)[None, :]
    live = r < counts[:, None]
    step = (span // counts.clamp(min=1)).to(torch.int32)[:, None]
    base = torch.arange(nb, dtype=torch.int64, device=DEV)[:, None] * be
    I = torch.where(live, r * step + (0 if multi else base.to(torch.int32)), -1)
    dt = torch.int16 if width == 2 else torch.uint8
    V = torch.randint(0, 1 << (8 * width - 1), (nb, be), generator=g, device=DEV, dtype=dt)
    where = ((r * step).to(torch.int64) + base)[live]
    return I, V, counts.to(torch.int32), where, V[live]


def cut(n):
    """Tensor sizes: 200 small ones (one bucket holds more segments than the cache), then large ones of odd sizes."""
    sizes = [9] * 200
    rest = n - sum(sizes)
    return sizes + [rest // 3 + 1, 7, rest - rest // 3 - 8]


@pytest.mark.parametrize("width", [2, 1])
@pytest.mark.parametrize("multi", [False, True])
@pytest.mark.parametrize("nb,be", CASES)
def test_apply_grouped(nb, be, multi, width):
    from paper_2605_07330_amd import srs
    print(f"case nb={nb} be={be} multi={multi} width={width}", flush=True)
    n = nb * be - be // 3
    I, V, counts, where, values = make_payload(nb, be, n, width, multi, nb + width)
    dt = torch.int16 if width == 2 else torch.uint8
    w = torch.randint(0, 120, (n,), device=DEV, dtype=dt)
    want = w.clone()
    want[where] = values
    ctx = srs.Context(0)
    try:
        def apply():
            if multi:
                sizes = cut(n)
                plan = ctx.plan(sizes, be)
                (ctx.apply_multi if width == 2 else ctx.apply_multi_u8)(plan, list(w.split(sizes)), I, V, counts, be)
                torch.cuda.synchronize()
                plan.close()
            else:
                (ctx.apply if width == 2 else ctx.apply_u8)(w, be, I, V, counts, be)
        apply()
        assert ctx.status() == 0
        assert torch.equal(w, want)
        # the last pair of the first bucket, deep in its groups, leaves the span: it alone is skipped, and reported
        last = int(counts[0]) - 1
        I[0, last] = be
        w[min(be, n) - 1] = 0
        want[min(be, n) - 1] = 0
        apply()
        assert ctx.status() == srs.FLAG_BAD_INDEX
        assert torch.equal(w[:be], want[:be]) and torch.equal(w, want)
    finally:
        ctx.close()


@pytest.mark.parametrize("width", [2, 1])
@pytest.mark.parametrize("multi", [False, True])
def test_second_pass_grouped(multi, width):
    """The refresh reads the snapshot pointers of a list out of the table of pairs; every third bucket has changed by half."""
    from paper_2605_07330_amd import srs
    nb, be = 1100, 33_000
    n = nb * be - 5
    dt = torch.int16 if width == 2 else torch.uint8
    old = torch.randint(0, 120, (n,), device=DEV, dtype=dt)
    heavy = (torch.arange(n, device=DEV) // be) % 3 == 0
    change = torch.rand(n, device=DEV) < torch.where(heavy, 0.5, 0.001)
    new = torch.where(change, old + 1, old)
    snap, roll = old.clone(), old.clone()
    alloc = srs.alloc_payload if width == 2 else srs.alloc_payload_u8
    I, V, counts = alloc(nb, be, DEV)
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_SNAPSHOT, 2)
        if multi:
            sizes = cut(n)
            plan = ctx.plan(sizes, be)
            ex, ap = (ctx.extract_multi, ctx.apply_multi) if width == 2 else (ctx.extract_multi_u8, ctx.apply_multi_u8)
            ex(plan, list(snap.split(sizes)), list(new.split(sizes)), I, V, counts, be)
            ap(plan, list(roll.split(sizes)), I, V, counts, be)
        else:
            ex, ap = (ctx.extract, ctx.apply) if width == 2 else (ctx.extract_u8, ctx.apply_u8)
            ex(snap, new, be, I, V, counts, be)
            ap(roll, be, I, V, counts, be)
        assert ctx.status() == 0
        full = torch.nn.functional.pad(change, (0, nb * be - n)).view(nb, be)
        assert torch.equal(counts[:nb].to(torch.int64), full.sum(dim=1))
        assert torch.equal(snap, new) and torch.equal(roll, new)
    finally:
        ctx.close()
