"""Batches of more than four items per CU, whose items are cut into one run per
XCD: every keyframe is updated as it is alone on the uncut grid, with a keyframe
that spans several runs, runs that hold many keyframes, and ragged ends."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from scenegen import make_keyframe, spec_for_config

pytestmark = pytest.mark.gpu

TINY = [(32, 24, 1), (20, 36, 3), (64, 48, 2), (16, 16, 1), (48, 20, 4)]


@pytest.mark.parametrize("sizes,patch,lam", [
    ([(640, 480, 5)] + TINY, 4, 0.0),                   # one keyframe over several runs, the rest in one
    (TINY + [(640, 480, 2)] + TINY, 4, 1e-3),
    ([(404, 300, 1 + 3 * i) for i in range(5)], 4, 0.0),
    ([(832, 628, 3), (840, 620, 1)], 16, 0.0),
    ([(340, 260, 2)] * 3 + TINY, 8, 0.0)])
def test_batch_equals_each_keyframe_alone(sizes, patch, lam):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        blocks = [-(-(w // patch) // (16 // patch)) * -(-(h // patch) // (16 // patch)) for w, h, _ in sizes]
        per_block = {4: 1, 8: 4, 16: 1}[patch]          # items of the plan below, before a form splits them
        assert sum(blocks) * per_block >= 4 * sg.sgn_device_info(0)["compute_units"]
        prm = sg.params(iters=3, lm_lambda=lam)
        base = dataclasses.replace(spec_for_config(1), n_rects=3, half_new=False, patch=patch)
        kfs = [make_keyframe(dataclasses.replace(base, width=w, height=h, n_nbr=n, seed=80 + i), device="cuda")
               for i, (w, h, n) in enumerate(s for s in sizes if s[0] >= patch and s[1] >= patch)]
        print(f"case large shares {sizes} {patch}x{patch} lambda {lam}", flush=True)
        grid = (4, 4) if patch == 4 else (1, 1)
        ds = [engine.DeviceKeyframe.from_scene(ctx, k) for k in kfs]
        engine.update_batch(ctx, ds, prm, sg.plan(*grid, 0, 0, 0, 1, groups=1))
        torch.cuda.synchronize()
        for d, k in zip(ds, kfs):
            a = engine.DeviceKeyframe.from_scene(ctx, k)
            engine.update_plain(ctx, a, prm, sg.plan(*grid, 0, 0, 0, 0, groups=1))
            torch.cuda.synchronize()
            got, want = d.state.to_host(), a.state.to_host()
            for f in want:
                assert np.array_equal(got[f], want[f]), f
            assert np.array_equal(d.inv_depth_out.cpu().numpy(), a.inv_depth_out.cpu().numpy())
    finally:
        ctx.close()
