"""Apply of payloads with well above 2048 chunk slots, most of them empty, against the oracle, tolerance 0: few pairs, full
buckets next to empty ones, 1024 buckets and one more, counts above cap, both element widths, single tensors and lists."""
import numpy as np
import pytest
import torch

import oracle
from util import from_u16, u16

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (buckets, bucket_elems, cap, kind): slots = buckets * ceil(min(cap, bucket_elems) / 2048)
CASES = [(1, 4_300_000, 4_300_000, "few"), (3, 1_500_000, 1_500_000, "few"), (33, 140_000, 140_000, "ends"),
         (700, 6_000, 6_000, "skew"), (1024, 4_097, 4_097, "ends"), (1025, 4_097, 4_097, "ends"), (1024, 4_200, 5_000, "none"),
         (64, 70_000, 66_000, "over"), (2, 2_200_000, 2_200_000, "rows")]


def make_counts(nb, be, cap, kind, rng):
    c = np.zeros(nb, np.int64)
    if kind == "few":
        c[:] = rng.integers(1, 5000, nb)
    elif kind == "ends":
        c[0] = c[-1] = min(be, 2049)
        c[nb // 2] = min(be, 4096)
    elif kind == "skew":
        c[:] = np.where(rng.random(nb) < 0.1, rng.integers(0, be + 1, nb), rng.integers(0, 3, nb))
    elif kind == "over":
        c[:] = rng.integers(0, 4000, nb)
        c[5], c[-1] = be, 0
    elif kind == "rows":                       # 1024 chunks and one more
        c[:] = [1024 * 2048, 1]
    return np.minimum(c, be)


@pytest.mark.parametrize("width", [2, 1])
@pytest.mark.parametrize("multi", [False, True])
@pytest.mark.parametrize("nb,be,cap,kind", CASES)
def test_apply_walk(nb, be, cap, kind, multi, width):
    from paper_2605_07330_amd import srs
    print(f"case nb={nb} be={be} cap={cap} kind={kind} multi={multi} width={width}", flush=True)
    rng = np.random.default_rng(nb + be + width)
    n = nb * be - be // 3
    counts = make_counts(nb, be, cap, kind, rng)
    counts[-1] = min(counts[-1], n - (nb - 1) * be)
    I = np.full((nb, cap), -1, np.int32)
    dt = np.uint16 if width == 2 else np.uint8
    V = np.zeros((nb, cap), dt)
    for b in range(nb):
        span = min(be, n - b * be)
        k = int(min(counts[b], cap))
        pos = np.sort(rng.choice(span, size=k, replace=False)) if k < span // 2 else np.arange(k)
        I[b, :k] = pos + (0 if multi else b * be)
        V[b, :k] = rng.integers(0, 1 << (8 * width), size=k)
    c32 = counts.astype(np.uint32)
    w = rng.integers(0, 1 << (8 * width), size=n, dtype=dt)
    cuts = [0, n // 5, n // 5 + 7, n // 2 + 1, n]
    sizes = [b - a for a, b in zip(cuts, cuts[1:])]
    want = [w[a:b].copy() for a, b in zip(cuts, cuts[1:])] if multi else w.copy()
    if multi:
        (oracle.apply_multi if width == 2 else oracle.apply_multi_u8)(want, sizes, be, I, V, c32)
        want = np.concatenate(want)
    else:
        (oracle.apply if width == 2 else oracle.apply_u8)(want, be, I, V, c32)
    d = from_u16(w, DEV) if width == 2 else torch.from_numpy(w.copy()).to(DEV)
    dI = torch.from_numpy(I).to(DEV)
    dV = torch.from_numpy(V.view(np.int16) if width == 2 else V).to(DEV)
    dc = torch.from_numpy(c32.view(np.int32)).to(DEV)
    ctx = srs.Context(0)
    try:
        if multi:
            plan = ctx.plan(sizes, be)
            parts = [d[a:b] for a, b in zip(cuts, cuts[1:])]
            (ctx.apply_multi if width == 2 else ctx.apply_multi_u8)(plan, parts, dI, dV, dc, cap)
        else:
            (ctx.apply if width == 2 else ctx.apply_u8)(d, be, dI, dV, dc, cap)
        assert ctx.status() == 0
    finally:
        ctx.close()
    got = u16(d) if width == 2 else d.cpu().numpy()
    assert np.array_equal(got, want)
