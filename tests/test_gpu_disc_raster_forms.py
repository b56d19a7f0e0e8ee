"""The disc raster's two splits of a tile, a wavefront with four pixels per lane
and four with one: keyframes rendered in a batch of many tiles equal each of them
alone, where few tiles with long lists take the other split."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.helpers import random_unit_cap
from tests.rules import lib

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(16, 16), (17, 35), (61, 14), (640, 480), (403, 799)])
def test_batch_render_equals_each_keyframe_alone(W, H):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        rng = np.random.default_rng(W)
        cus = sg.sgn_device_info(0)["compute_units"]
        tiles = -(-W // 16) * -(-H // 16)
        img = torch.zeros((H, W), dtype=torch.float32)
        dks = []
        for m, r in ((10 * tiles, 5.0), (30 * tiles, 12.0), (16 * tiles, 3.3)):
            m += m % 2
            assert lib().raster_pixels(tiles, m / tiles * lib().mean_tiles(r, 16), cus) == (1 if tiles <= 5 * cus else 4)
            u = rng.uniform(-4, [W + 4, H + 4], (m, 2))
            ns = np.array([random_unit_cap(rng, 50) for _ in range(m)], np.float32)
            idp = rng.uniform(0.2, 2.0, m)
            u[1::2], ns[1::2], idp[1::2] = u[::2], ns[::2], idp[::2]          # ties
            dks.append(engine.DiscKeyframe(ctx, img, img[None], np.eye(3)[None], np.zeros((1, 3)),
                                           (0.9 * W, 0.9 * W, W / 2, H / 2), r, u[:, 0], u[:, 1], idp, ns))
        print(f"case disc raster {W}x{H}", flush=True)
        # the batch is brought above the line by an empty keyframe's tiles
        side = 16 * (int((5 * cus) ** 0.5) + 1)
        big = torch.zeros((side, side), dtype=torch.float32)
        dks.append(engine.DiscKeyframe(ctx, big, big[None], np.eye(3)[None], np.zeros((1, 3)),
                                       (side, side, side / 2, side / 2), 5.0, np.full(1, -99.0), np.zeros(1),
                                       np.ones(1), np.array([[0, 0, -1]], np.float32)))
        engine.disc_render(ctx, dks)
        torch.cuda.synchronize()
        got = [(d.inv_depth_out.clone(), d.index_out.clone()) for d in dks[:-1]]
        for d, (depth, index) in zip(dks, got):
            d.inv_depth_out.fill_(7.0)
            d.index_out.fill_(7)
            d.render()
            torch.cuda.synchronize()
            assert torch.equal(d.index_out, index) and torch.equal(d.inv_depth_out, depth)
            drawn = index[index >= 0]
            assert drawn.numel() > 0 and not bool((drawn % 2 == 1).any())
    finally:
        ctx.close()
