"""The forms of the Gauss-Newton kernel that a batch's size picks (columns
split over lanes, one or two frames in flight, one sample at a time) and the
bounded persistent grid: one keyframe's result is bitwise the same in each."""
import dataclasses

import numpy as np
import pytest

torch = pytest.importorskip("torch")

from scenegen import make_keyframe, spec_for_config

pytestmark = pytest.mark.gpu

FIELDS = ("inv_depth", "nx", "ny", "nz", "flags", "cost", "nvalid", "last_update")


@pytest.mark.parametrize("storage,patch,lam,n_nbr", [
    ("f16", 4, 0.0, 7), ("f32", 4, 0.0, 3), ("u8", 4, 0.0, 1), ("f16", 4, 1e-3, 5), ("u8", 4, 1e-3, 16), ("f32", 4, 1e-3, 2),
    ("f32", 16, 0.0, 5),
    ("u8", 16, 1e-3, 2), ("f16", 16, 0.0, 4), ("f16", 8, 0.0, 5)])
def test_every_form_gives_one_result(storage, patch, lam, n_nbr):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        # ragged in both directions: 300 anchor blocks, the last ones partly outside the grid
        spec = dataclasses.replace(spec_for_config(1), width=308, height=234, n_rects=6, seed=23, patch=patch,
                                   n_nbr=n_nbr, half_new=False)
        kf = make_keyframe(spec, device="cuda")
        prm = sg.params(iters=4, lm_lambda=lam)
        base = engine.DeviceKeyframe.from_scene(ctx, kf, storage=storage, render=False)
        ref = None
        # items per SIMD: 0.3, 1.2, 2.6, 5.9, 26; then the persistent grid
        runs = [(1, None), (4, None), (9, None), (20, None), (90, None)]
        grid = (4, 4) if patch == 4 else (1, 1)
        runs += [(20, sg.plan(*grid, 1, 8, 0, 1, groups=1)), (2, sg.plan(*grid, 1, 4, 0, 0, groups=1))]
        for k, plan in runs:
            print(f"case {storage} {patch}x{patch} lambda {lam}: {k} copies, "
                  f"{'default' if plan is None else 'persistent'}", flush=True)
            states = [base.state.clone() for _ in range(k)]
            items = sg.batch_array([sg.sgn_batch_item(base.view.c, s.c, None, None, None) for s in states])
            sg.sgn_optimize_batch(ctx.handle, items, k, prm, plan)
            torch.cuda.synchronize()
            for s in states:
                got = [getattr(s, f).view(torch.int32) for f in FIELDS]
                if ref is None:
                    ref = got
                    assert int((s.nvalid > 0).sum()) > 0.8 * s.nvalid.numel()
                for f, a, b in zip(FIELDS, got, ref):
                    assert torch.equal(a, b), (k, f, int((a != b).sum()))
    finally:
        ctx.close()


def test_full_keyframe_equals_its_default_and_four_group_plans_for_8x8():
    """8 x 8 surfels: the default plan of a small keyframe (one group per
    wavefront) against the explicit four-group plan."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        kf = make_keyframe(spec_for_config(0), device="cuda")
        out = []
        for plan in (None, sg.plan(1, 1, 0, 0, 0, 1, groups=4)):
            d = engine.DeviceKeyframe.from_scene(ctx, kf)
            engine.update_plain(ctx, d, sg.params(iters=6), plan)
            torch.cuda.synchronize()
            out.append(d.state.to_host())
        for f in out[0]:
            assert np.array_equal(out[0][f], out[1][f]), f
    finally:
        ctx.close()


@pytest.mark.parametrize("storage,lam,n_nbr,radius", [
    ("f16", 0.0, 6, 10.0), ("f32", 0.0, 3, 10.0), ("u8", 0.0, 1, 2.5), ("f16", 1e-3, 5, 10.0),
    ("f32", 0.0, 16, 12.0), ("f16", 0.0, 16, 12.0)])
def test_every_disc_form_gives_one_result(storage, lam, n_nbr, radius):
    """Disc surfels: copies of one keyframe take the batch through every form
    (sixteen, eight, four or one wavefronts per item, taps of four, two or no
    frames ahead, solves shared or not).  An odd count leaves half an item
    empty; some discs are cut by the image border."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    from scenegen import make_disc_surfels
    ctx = sg.Context(0)
    try:
        spec = dataclasses.replace(spec_for_config(1), width=308, height=234, n_rects=6, seed=29, n_nbr=n_nbr,
                                   half_new=False)
        kf = make_keyframe(spec, device="cuda")
        d = engine.DiscKeyframe.from_scene(ctx, kf, make_disc_surfels(kf, radius=radius), storage=storage)
        d.count -= 1 - d.count % 2
        m = d.count
        per = (m + 1) // 2 if storage != "f32" else m
        prm = sg.params(iters=3, lm_lambda=lam)
        simds = 4 * sg.sgn_device_info(0)["compute_units"]
        ref = None
        for w in (0.1, 0.35, 0.8, 1.5, 2.0, 3.0, 4.5, 5.5, 7.0, 12.0):
            k = max(1, int(w * simds / per))
            print(f"case discs {storage} lambda {lam}: {k} copies of {m}, {k * per / simds:.2f} items per SIMD", flush=True)
            states = [d.state.clone() for _ in range(k)]
            items = sg.disc_array([sg.sgn_disc_item(d.img.view.c, s.c, d.ux.data_ptr(), d.uy.data_ptr(), m, radius)
                                   for s in states])
            sg.sgn_disc_optimize(ctx.handle, items, k, prm)
            torch.cuda.synchronize()
            for s in states:
                got = [getattr(s, f).view(torch.int32) for f in FIELDS]
                if ref is None:
                    ref = got
                    assert int((s.nvalid[:m] > 0).sum()) > 0.8 * m
                for f, a, b in zip(FIELDS, got, ref):
                    assert torch.equal(a, b), (k, f, int((a != b).sum()))
    finally:
        ctx.close()
