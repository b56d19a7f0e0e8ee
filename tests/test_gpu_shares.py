"""Work items cut into one run per XCD: every keyframe of a batch is updated
as it is alone, whatever the number of keyframes and their sizes (runs that
end inside a keyframe, runs with no item, keyframes with no surfel)."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from scenegen import make_disc_surfels, make_keyframe, spec_for_config

pytestmark = pytest.mark.gpu


def _specs(sizes):
    base = dataclasses.replace(spec_for_config(1), n_rects=3, half_new=False)
    return [dataclasses.replace(base, width=w, height=h, n_nbr=n, seed=40 + i) for i, (w, h, n) in enumerate(sizes)]


@pytest.mark.parametrize("sizes", [
    [(16, 16, 1)], [(20, 36, 3), (64, 48, 2)], [(160, 120, 12), (64, 48, 1), (32, 32, 4)],
    [(64 + 16 * i, 48 + 4 * i, 1 + i % 5) for i in range(9)]])
def test_tile_batch_equals_each_keyframe_alone(sizes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        prm = sg.params(iters=3)
        kfs = [make_keyframe(s, device="cuda") for s in _specs(sizes)]
        ds = [engine.DeviceKeyframe.from_scene(ctx, k) for k in kfs]
        print(f"case tile shares {sizes}", flush=True)
        engine.update_batch(ctx, ds, prm)
        torch.cuda.synchronize()
        for d, k in zip(ds, kfs):
            a = engine.DeviceKeyframe.from_scene(ctx, k)
            engine.update_plain(ctx, a, prm, sg.plan(4, 4, 0, 0, 0, 0, groups=1))
            torch.cuda.synchronize()
            got, want = d.state.to_host(), a.state.to_host()
            for f in want:
                assert np.array_equal(got[f], want[f]), f
            assert np.array_equal(d.inv_depth_out.cpu().numpy(), a.inv_depth_out.cpu().numpy())
    finally:
        ctx.close()


@pytest.mark.parametrize("storage,counts", [("f16", [1]), ("f32", [3, 1]), ("f16", [17, 0, 5]),
                                            ("u8", [9, 2, 0, 31, 1, 8, 4, 12, 3])])
def test_disc_batch_equals_each_keyframe_alone(storage, counts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        prm = sg.params(iters=3)
        kfs = [make_keyframe(s, device="cuda") for s in _specs([(128, 96, 1 + i % 4) for i in range(len(counts))])]
        sets = [make_disc_surfels(k, radius=10.0) for k in kfs]

        def build(i):
            d = engine.DiscKeyframe.from_scene(ctx, kfs[i], sets[i], storage=storage)
            d.count = min(counts[i], d.count)
            return d
        ds = [build(i) for i in range(len(kfs))]
        print(f"case disc shares {storage} {counts}", flush=True)
        engine.disc_update(ctx, ds, prm)
        torch.cuda.synchronize()
        for i, d in enumerate(ds):
            a = build(i)
            if a.count:
                engine.disc_update(ctx, [a], prm)
            torch.cuda.synchronize()
            got, want = d.state.to_host(), a.state.to_host()
            for f in want:
                assert np.array_equal(got[f], want[f]), (i, f)
    finally:
        ctx.close()
