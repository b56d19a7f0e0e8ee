"""Disc renders on both sides of the line between binning a keyframe in one
workgroup and over the device: a batch of twelve keyframes (in LDS to 6,400
discs each) equals each of them alone (in LDS to 3,072)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from tests.helpers import random_unit_cap

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("most", [3073, 6400, 6401])
def test_batch_render_equals_each_keyframe_alone(most):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        rng = np.random.default_rng(most)
        W, H = 360, 250
        ns = np.array([random_unit_cap(rng, 50) for _ in range(most)], np.float32)
        counts = [most, 0, 1, 63, 64, 65, 300, 3072, 3073, 1000, 2, 500]
        print(f"case disc bin lines, twelve keyframes, at most {most} discs", flush=True)
        img = torch.zeros((H, W), dtype=torch.float32)
        dks = []
        for m in counts:
            d = engine.DiscKeyframe(ctx, img, img[None], np.eye(3)[None], np.zeros((1, 3)),
                                    (0.9 * W, 0.9 * W, W / 2, H / 2), 6.0, rng.uniform(-4, W + 4, max(m, 1)),
                                    rng.uniform(-4, H + 4, max(m, 1)), rng.uniform(0.2, 2.0, max(m, 1)), ns[:max(m, 1)])
            d.count = m
            dks.append(d)
        engine.disc_render(ctx, dks)
        torch.cuda.synchronize()
        got = [(d.inv_depth_out.clone(), d.index_out.clone()) for d in dks]
        for d, (depth, index) in zip(dks, got):
            d.inv_depth_out.fill_(7.0)
            d.index_out.fill_(7)
            d.render()
            torch.cuda.synchronize()
            assert torch.equal(d.index_out, index), d.count
            assert torch.equal(d.inv_depth_out, depth), d.count
        assert int((got[0][1] >= 0).sum()) > 0.9 * W * H and int((got[1][1] >= 0).sum()) == 0
    finally:
        ctx.close()
