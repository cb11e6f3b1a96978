"""Single one-byte tensors on either side of the sizes where the number of tiles in a bucket makes the library pick the next
tile, the bucket as large as the tensor, larger and half of it; against the oracle, tolerance 0."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("mode", [0, 1, 2])
@pytest.mark.parametrize("tile", [8192, 16384])
def test_tiles_of_one_byte_elements(tile, mode):
    from paper_2605_07330_amd import srs
    ctx = srs.Context(0)
    try:
        ctx.set_option(srs.OPT_SNAPSHOT, mode)
        for n in (192 * tile - 1, 192 * tile, 192 * tile + 1):
            for be in (n, 2 * n, n // 2 + 1):
                print(f"case tile={tile} mode={mode} n={n} be={be}", flush=True)
                rng = np.random.default_rng(n + be)
                old = rng.integers(0, 256, n).astype(np.uint8)
                change = rng.random(n) < 0.003
                change[[0, -1]] = True
                new = np.where(change, ~old, old).astype(np.uint8)
                cap = min(be, 40_000)
                after = old.copy()
                wI, wV, wc, overflow = oracle.extract_u8(after, new, be, cap)
                t, u = torch.from_numpy(old.copy()).to(DEV), torch.from_numpy(new).to(DEV)
                I, V, counts = srs.alloc_payload_u8(len(wc), cap, DEV)
                ctx.extract_u8(t, u, be, I, V, counts, cap)
                assert ctx.status() == 0 and not overflow
                assert np.array_equal(counts.cpu().numpy().view(np.uint32)[:len(wc)], wc)
                live = np.arange(cap)[None, :] < wc[:, None]
                gI, gV = I.cpu().numpy().reshape(len(wc), cap), V.cpu().numpy().reshape(len(wc), cap)
                assert np.array_equal(gI[live], wI[live]) and np.array_equal(gV[live], wV[live])
                assert np.array_equal(t.cpu().numpy(), old if mode == 1 else after)
    finally:
        ctx.close()
