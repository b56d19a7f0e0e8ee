"""Images whose last byte is the last of their memory: f16 and u8 taps come as
aligned eight-byte words, which must not read the dword past it.  The update
equals, bitwise, the one on the same images with memory behind them."""
import dataclasses

import pytest

torch = pytest.importorskip("torch")

from scenegen import make_disc_surfels, make_keyframe, spec_for_config

pytestmark = pytest.mark.gpu

MB = 1 << 20
FIELDS = ("inv_depth", "nx", "ny", "nz", "flags", "cost", "nvalid", "last_update")


def _at_end_of_memory(images, pitch):
    """The images copied to rows of `pitch` elements of which the last ends
    with its width, at the end of a memory segment."""
    k, h, w = images.shape
    n, size = (((k * h) - 1) * pitch + w) * images.element_size(), 12 * MB
    assert n <= size
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    kept = []                             # until the free blocks of other segments are used up
    for _ in range(32):
        buf = torch.empty(size, dtype=torch.uint8, device="cuda")
        if any(buf.data_ptr() + size == s["address"] + s["total_size"] for s in torch.cuda.memory_snapshot()):
            break
        kept.append(buf)
    else:
        raise AssertionError("no allocation ends its segment")
    out = buf[size - n:].view(images.dtype).as_strided((k, h, w), (h * pitch, pitch, 1))
    out.copy_(images)
    return out


@pytest.mark.parametrize("storage", ["f16", "u8"])
@pytest.mark.parametrize("disc,lam,pad", [(False, 0.0, 0), (False, 1e-3, 0), (True, 0.0, 0), (False, 0.0, 16),
                                          (False, 1e-3, 64), (True, 0.0, 16)])
def test_images_at_the_end_of_their_memory(storage, disc, lam, pad):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import engine, surfgn as sg
    ctx = sg.Context(0)
    try:
        spec = dataclasses.replace(spec_for_config(1), n_nbr=3, half_new=False, seed=31)
        kf = make_keyframe(spec, device="cuda")
        prm = sg.params(iters=8, lm_lambda=lam)
        got = []
        for end in (False, True):
            print(f"case image end {storage} disc {disc} lambda {lam} pitch + {pad} at the end {end}", flush=True)
            if disc:
                d = engine.DiscKeyframe.from_scene(ctx, kf, make_disc_surfels(kf, radius=10.0), storage=storage)
                img = d.img
            else:
                d = img = engine.DeviceKeyframe.from_scene(ctx, kf, storage=storage, render=False)
            if end:
                img.nbr_imgs = _at_end_of_memory(img.nbr_imgs, img.width + pad)
                img.view = sg.KeyframeView(img.kf_img, [img.nbr_imgs[i] for i in range(img.n_nbr)], img.R, img.t,
                                           img.K, img.patch, img.scale)
            if disc:
                engine.disc_update(ctx, [d], prm)
            else:
                engine.update_plain(ctx, d, prm)
            torch.cuda.synchronize()
            got.append([getattr(d.state, f).view(torch.int32).clone() for f in FIELDS])
        for f, a, b in zip(FIELDS, *got):
            assert torch.equal(a, b), f
        assert int((got[0][6] > 0).sum()) > 0.8 * got[0][6].numel()
    finally:
        ctx.close()
