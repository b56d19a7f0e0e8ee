"""Neighbour images with rows of 16 KiB and more are read by byte offset: every
form of the tile and disc kernels that a batch's size picks gives, bitwise, the
result of the same images in narrow rows."""
import dataclasses

import pytest

torch = pytest.importorskip("torch")

from scenegen import make_disc_surfels, make_keyframe, spec_for_config

pytestmark = pytest.mark.gpu

FIELDS = ("inv_depth", "nx", "ny", "nz", "flags", "cost", "nvalid", "last_update")


def _wide(sg, dk):
    pitch = 16384 // dk.nbr_imgs.element_size() + 4
    wide = torch.zeros((dk.n_nbr, dk.height, pitch), dtype=dk.nbr_imgs.dtype, device="cuda")
    wide[:, :, :dk.width] = dk.nbr_imgs
    return sg.KeyframeView(dk.kf_img, [wide[i, :, :dk.width] for i in range(dk.n_nbr)], dk.R, dk.t, dk.K, dk.patch,
                           dk.scale)


def _words(s):
    return [getattr(s, f).view(torch.int32) for f in FIELDS]


@pytest.mark.parametrize("storage,patch,lam", [
    ("f16", 4, 0.0), ("f32", 4, 0.0), ("u8", 4, 0.0), ("f16", 4, 1e-3), ("u8", 4, 1e-3), ("f32", 16, 0.0),
    ("u8", 16, 0.0), ("f16", 16, 1e-3), ("u8", 8, 0.0)])
def test_tile_forms(storage, patch, lam):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        spec = dataclasses.replace(spec_for_config(1), width=308, height=234, n_rects=6, seed=47, patch=patch, n_nbr=3,
                                   half_new=False)
        d = engine.DeviceKeyframe.from_scene(ctx, make_keyframe(spec, device="cuda"), storage=storage, render=False)
        wide, prm, want = _wide(sg, d), sg.params(iters=4, lm_lambda=lam), None
        # 300 items each (8x8 surfels 1,102): 0.3, 1.2, 2.6, 5.9 and 26 per SIMD
        for k, view in [(1, d.view)] + [(k, wide) for k in (1, 4, 9, 20, 90)]:
            print(f"case wide rows {storage} {patch}x{patch} lambda {lam}: {k} copies, "
                  f"{'narrow' if view is d.view else 'wide'}", flush=True)
            states = [d.state.clone() for _ in range(k)]
            items = sg.batch_array([sg.sgn_batch_item(view.c, s.c, None, None, None) for s in states])
            sg.sgn_optimize_batch(ctx.handle, items, k, prm, None)
            torch.cuda.synchronize()
            want = want or _words(states[0])
            for s in states:
                for f, a, b in zip(FIELDS, _words(s), want):
                    assert torch.equal(a, b), (k, f)
        assert int((want[6] > 0).sum()) > 0.8 * want[6].numel()
    finally:
        ctx.close()


@pytest.mark.parametrize("storage,lam", [("f16", 0.0), ("f32", 0.0), ("u8", 0.0), ("f16", 1e-3), ("f32", 1e-3)])
def test_disc_forms(storage, lam):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        spec = dataclasses.replace(spec_for_config(1), width=308, height=234, n_rects=6, seed=53, n_nbr=3,
                                   half_new=False)
        kf = make_keyframe(spec, device="cuda")
        d = engine.DiscKeyframe.from_scene(ctx, kf, make_disc_surfels(kf, radius=10.0), storage=storage)
        wide, prm, want, m = _wide(sg, d.img), sg.params(iters=3, lm_lambda=lam), None, d.count
        per = (m + 1) // 2 if storage != "f32" else m
        simds = 4 * sg.sgn_device_info(0)["compute_units"]
        # the lines of the forms: items per SIMD
        for w, view in [(0.1, d.img.view)] + [(w, wide) for w in (0.1, 0.4, 0.9, 1.9, 3.0, 4.6, 5.5, 7.0, 9.0)]:
            k = max(1, round(w * simds / per))
            print(f"case wide rows discs {storage} lambda {lam}: {k} copies of {m}", flush=True)
            states = [d.state.clone() for _ in range(k)]
            items = sg.disc_array([sg.sgn_disc_item(view.c, s.c, d.ux.data_ptr(), d.uy.data_ptr(), m, 10.0)
                                   for s in states])
            sg.sgn_disc_optimize(ctx.handle, items, k, prm)
            torch.cuda.synchronize()
            want = want or _words(states[0])
            for s in states:
                for f, a, b in zip(FIELDS, _words(s), want):
                    assert torch.equal(a, b), (k, f)
        assert int((want[6][:m] > 0).sum()) > 0.8 * m
    finally:
        ctx.close()
