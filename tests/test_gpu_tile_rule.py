"""Single tensors at the sizes where the library takes another tile: by the number of tiles in a bucket, by their number in all, and
buckets that one tile just holds; many small buckets; against the oracle, tolerance 0."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EDGES = [(128 * 4096, 1), (256 * 8192, 1), (256 * 16384, 1), (768 * 4096, 8), (768 * 8192, 6), (768 * 16384, 6), (8192, 1), (3 * 8192, 3),
         (300 * 4096, 300), (1000 * 8192, 1000), (900 * 8200, 900), (800 * 16384, 800), (10 * 16384, 10)]


@pytest.mark.parametrize("kind", ["bf16", "cast", "u8"])
@pytest.mark.parametrize("n,nb", EDGES)
def test_around_the_lines_of_the_rule(n, nb, kind):
    from paper_2605_07330_amd import srs
    ctx = srs.Context(0)
    try:
        for be in (n // nb - 1, n // nb, n // nb + 1):
            print(f"case {kind} n={n} be={be}", flush=True)
            rng = np.random.default_rng(be)
            dt = np.uint8 if kind == "u8" else np.uint16
            mask = rng.random(n) < 0.003
            mask[[0, -1]] = True
            if kind == "cast":
                new = (rng.standard_normal(n) * 0.02).astype(np.float32)
                old = (oracle.round_bf16(new) ^ mask).astype(np.uint16)
            else:
                old = rng.integers(0, 1 << (8 * dt().itemsize), n).astype(dt)
                new = (old ^ mask).astype(dt)
            cap = min(be, n // nb // 50 + 200)
            after = old.copy()
            fn = {"bf16": oracle.extract, "u8": oracle.extract_u8, "cast": oracle.extract_cast}[kind]
            wI, wV, wc = fn(after, new, be, cap)[:3]
            as_torch = lambda a: torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).to(DEV)  # noqa: E731
            t, u = as_torch(old.copy()), as_torch(new)
            I, V, counts = (srs.alloc_payload_u8 if kind == "u8" else srs.alloc_payload)(len(wc), cap, DEV)
            {"bf16": ctx.extract, "u8": ctx.extract_u8, "cast": ctx.extract_cast}[kind](t, u, be, I, V, counts, cap)
            assert ctx.status() == 0
            assert np.array_equal(counts.cpu().numpy().view(np.uint32)[:len(wc)], wc)
            live = np.arange(cap)[None, :] < np.asarray(wc)[:, None]
            gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().view(dt).reshape(len(wc), cap)
            assert np.array_equal(gI[live], wI[live]) and np.array_equal(gV[live], wV[live])
            assert np.array_equal(t.cpu().numpy().view(dt), after)
    finally:
        ctx.close()
