"""Image storage where rows allow no wide loads and run over several
wavefronts: pixels 64 apart per thread, the last ones partly outside."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "u8"])
@pytest.mark.parametrize("W,H,src_pitch,dst_pitch", [
    (511, 5, 511, 511), (512, 3, 513, 512), (513, 6, 513, 513), (577, 4, 579, 577), (1023, 9, 1023, 1025),
    (1100, 7, 1101, 1103)])
def test_odd_rows(dtype, W, H, src_pitch, dst_pitch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1910_01997_amd import surfgn as sg
    ctx = sg.Context(0)
    try:
        gen = torch.Generator().manual_seed(W)
        src = torch.rand((H, src_pitch), generator=gen) * 1.4 - 0.2
        tdt = torch.float16 if dtype == "f16" else torch.uint8
        out = torch.full((H, dst_pitch), 77, dtype=tdt, device="cuda")
        scale = 1.0 if dtype == "f16" else 1.0 / 255.0
        dev = src.cuda()
        print(f"case quantize odd rows {dtype} {W}x{H} pitches {src_pitch} {dst_pitch}", flush=True)
        sg.sgn_quantize(ctx.handle, dev.data_ptr(), src_pitch,
                        sg.sgn_image(out.data_ptr(), W, H, dst_pitch, sg.SGN_F16 if dtype == "f16" else sg.SGN_U8,
                                     scale))
        torch.cuda.synchronize()
        x = src[:, :W]
        want = x.half() if dtype == "f16" else torch.round(x / torch.tensor(scale, dtype=torch.float32)).clamp(
            0, 255).to(tdt)
        got = out.cpu()
        assert torch.equal(got[:, :W], want)
        assert (got[:, W:] == 77).all()
    finally:
        ctx.close()
