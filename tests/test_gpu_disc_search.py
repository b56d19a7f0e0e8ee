"""The search for empty areas against the oracle where one pixel decides: few
owned pixels, so that every position of a window's scan (its first 64 pixels,
the rounds of 256 behind them, a ragged end) is the only one for some
candidate."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle

pytestmark = pytest.mark.gpu


# windows of 1, 9, 49, 81, 289, 361 and 1,089 pixels
@pytest.mark.parametrize("radius", [0.5, 1.0, 3.5, 4.0, 8.5, 9.0, 16.0])
def test_search_matches_oracle_on_sparse_maps(radius):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        W, H = 333, 217
        print(f"case disc search, radius {radius}", flush=True)
        rng = np.random.default_rng(int(radius * 10))
        img = torch.zeros((H, W), dtype=torch.float32)
        n = np.tile(np.float32([0, 0, -1]), (1, 1))
        alpha = 1.0 if radius <= 12 else 2.0
        for spacing in (2, 7):
            dk = engine.DiscKeyframe(ctx, img, img[None], np.eye(3)[None], np.zeros((1, 3)),
                                     (0.9 * W, 0.9 * W, W / 2, H / 2), radius / alpha, np.float32([5.0]), np.float32([5.0]),
                                     np.float32([1.0]), n, capacity=1 + (W // spacing + 1) * (H // spacing + 1))
            imap = np.where(rng.random((H, W)) < 0.7 / (np.pi * radius * radius + 1), 0, -1).astype(np.int32)
            dk.index_out.copy_(torch.from_numpy(imap).to(dk.index_out.device).view_as(dk.index_out))
            placed, found = dk.place(alpha=alpha, beta=alpha, spacing=spacing)
            xs, ys, want = oracle.disc_search(imap, radius / alpha, alpha, spacing)
            lattice = len(range(spacing // 2, W, spacing)) * len(range(spacing // 2, H, spacing))
            assert 0.2 * lattice < want < 0.95 * lattice
            assert placed == found == want
            ux, uy = dk.centres()
            assert np.array_equal(ux[1:], xs.astype(np.float32)) and np.array_equal(uy[1:], ys.astype(np.float32))
    finally:
        torch.cuda.synchronize()
        ctx.close()
