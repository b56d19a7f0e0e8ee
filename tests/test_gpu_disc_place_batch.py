"""Placement in batches about the sixteen keyframes that travel in the kernels'
arguments, with neighbour windows on both sides of two pixels per lane (121 and
169 pixels): each keyframe as it is alone."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.helpers import random_unit_cap

pytestmark = pytest.mark.gpu

FIELDS = ("inv_depth", "nx", "ny", "nz", "flags", "cost", "nvalid", "last_update")


@pytest.mark.parametrize("n", [2, 16, 17])
@pytest.mark.parametrize("radii", [(1.5, 2.5), (2.5, 2.6), (0.6, 10.0)])
def test_batch_placement_equals_each_keyframe_alone(n, radii):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        rng = np.random.default_rng(n)
        print(f"case placement of {n} keyframes, radii {radii}", flush=True)

        def make(i, seed):
            g = np.random.default_rng(seed)
            W, H, r = 40 + 9 * i, 70 - 3 * i, radii[1 if i == n // 2 else 0]
            m = int(0.5 * W * H / (3.2 * r * r)) + 1
            u = g.uniform(0, [W, 0.6 * H], (m, 2))                 # the lower part stays empty
            ns = np.array([random_unit_cap(g, 30) for _ in range(m)], np.float32)
            img = torch.zeros((H, W), dtype=torch.float32)
            d = engine.DiscKeyframe(ctx, img, img[None], np.eye(3)[None], np.zeros((1, 3)),
                                    (0.9 * W, 0.9 * W, W / 2, H / 2), r, u[:, 0], u[:, 1], g.uniform(0.2, 2.0, m), ns,
                                    capacity=m + W * H // (5 if i % 3 else 40))      # room for all or some
            d.render()
            return d
        seeds = rng.integers(0, 1 << 30, n)
        batch = [make(i, int(s)) for i, s in enumerate(seeds)]
        got = engine.disc_place(ctx, batch, spacing=3)
        placed = 0
        for i, (d, s) in enumerate(zip(batch, seeds)):
            a = make(i, int(s))
            assert a.place(spacing=3) == got[i] and a.count == d.count
            for f in FIELDS:
                assert torch.equal(getattr(a.state, f)[:a.count].view(torch.int32),
                                   getattr(d.state, f)[:a.count].view(torch.int32)), f
            assert torch.equal(a.ux[:a.count], d.ux[:a.count]) and torch.equal(a.uy[:a.count], d.uy[:a.count])
            placed += got[i][0]
        assert placed > 20 * n
    finally:
        ctx.close()
