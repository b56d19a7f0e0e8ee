"""The disc render's two ways of binning (a keyframe per workgroup in LDS, or
passes over the batch) and its depth test by products, against the oracle's
plain double walk: exact index maps and depths."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from tests.helpers import random_unit_cap
from tests.parity import oracle_keyframe, oracle_state

pytestmark = pytest.mark.gpu


def _surfels(rng, m, W, H):
    ux = rng.uniform(-6, W + 6, m).astype(np.float32)
    uy = rng.uniform(-6, H + 6, m).astype(np.float32)
    ids = rng.uniform(0.2, 2.0, m).astype(np.float32)
    ns = np.array([random_unit_cap(rng, 60) for _ in range(m)], np.float32)
    return ux, uy, ids, ns


@pytest.mark.parametrize("W,H,m", [
    (48, 33, 40),               # one ragged row of tiles
    (640, 400, 16384),          # the most surfels of the LDS form, 300 on a tile
    (640, 400, 16385),          # one more: passes over the batch
    (3072, 1280, 900),          # 15,360 tiles: the most of the LDS form
    (3088, 1280, 900),          # one column of tiles more
])
def test_bins_and_ties_match_the_oracle(W, H, m):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        rng = np.random.default_rng(W + m)
        ux, uy, ids, ns = _surfels(rng, m, W, H)
        # exact ties: the same plane and centre at another index; equal planes
        # (one inverse depth, facing the camera) at several centres
        k = min(m // 4, 60)
        ux[m - k:], uy[m - k:], ids[m - k:], ns[m - k:] = ux[:k], uy[:k], ids[:k], ns[:k]
        ids[k:2 * k], ns[k:2 * k] = 1.25, np.float32([0, 0, -1])
        # depths at the ends of float's range, not drawn, and beyond it
        ids[2 * k:2 * k + 5] = np.float32([1e-38, 3e38, -0.5, 0.0, np.inf])
        flags = np.zeros(m, np.uint32)
        flags[::17] = oracle.UNINIT
        print(f"case disc bins {W}x{H}, {m} discs", flush=True)
        img = torch.zeros((H, W), dtype=torch.float32)
        dk = engine.DiscKeyframe(ctx, img, img[None], np.eye(3)[None], np.zeros((1, 3)),
                                 (0.9 * W, 0.9 * W, W / 2, H / 2), 10.0, ux, uy, ids, ns, flags=flags)
        dk.render()
        torch.cuda.synchronize()
        idm, ind = oracle.disc_render(oracle_keyframe(dk), oracle_state(ids, ns, flags), ux.astype(np.float64),
                                      uy.astype(np.float64), 10.0)
        assert np.array_equal(dk.index_out.cpu().numpy(), ind)
        assert np.array_equal(dk.inv_depth_out.cpu().numpy(), idm.astype(np.float32))
        assert (ind >= 0).any()
    finally:
        ctx.close()
