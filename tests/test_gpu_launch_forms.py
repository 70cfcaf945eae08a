"""The same image through every form of launch that the rules choose between:
bands of 1 to 8 steps (SOBEL4X5_U8_WAVES), batches in bands of 4 to 256 rows on
either kind of grid, images in kernel arguments, tables in the fixed buffer.
All equal the oracle, call after call."""
import numpy as np
import pytest

from paper_2305_00515_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 3), (17, 63), (65, 127), (20, 257), (333, 700)]


@pytest.mark.parametrize("waves", ["", "1", "7", "64", "1000000"])
def test_single_images(oracle_mod, sobel_lib, gpu, monkeypatch, waves):
    monkeypatch.setenv("SOBEL4X5_U8_WAVES", waves)
    w = sobel_lib.family_weights(1, 3, 5, 10, 15, 30)
    for h, wd in SIZES + [(1080, 1920)]:
        img = synth.field_image(h, wd, h) if h * wd > 64 else synth.rect_image(h, wd, h)
        src = torch.from_numpy(img).to(gpu)
        for border in (0, 3):
            want = oracle_mod.sobel_u8(img, border)
            want_w = oracle_mod.sobel_u8(img, border, weights=w, want_dir=False)[0]
            for _ in range(2):
                mag = sobel_lib.sobel4x5_u8(src, border)[0]
                both, dirs = sobel_lib.sobel4x5_u8(src, border, dir_type=1)
                mag_w = sobel_lib.sobel4x5_u8_weighted(src, w, border)[0]
                torch.cuda.synchronize()
                assert np.array_equal(mag.cpu().numpy(), want[0]) and np.array_equal(both.cpu().numpy(), want[0])
                assert np.array_equal(np.stack([d.cpu().numpy() for d in dirs]), want[1])
                assert np.array_equal(mag_w.cpu().numpy(), want_w)


@pytest.mark.parametrize("static", ["0", "1"])
@pytest.mark.parametrize("th", ["4", "8", "16", "64", "256"])
def test_batches(oracle_mod, sobel_lib, gpu, monkeypatch, static, th):
    monkeypatch.setenv("SOBEL4X5_BATCH_TH", th)
    monkeypatch.setenv("SOBEL4X5_BATCH_STATIC", static)
    imgs = [synth.rect_image(h, w, h + w) % 7 for h, w in SIZES]
    srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
    want = [oracle_mod.sobel_u8(m) for m in imgs]
    for _ in range(2):
        outs = sobel_lib.sobel4x5_batched(srcs), sobel_lib.sobel4x5_batched_noalloc(srcs)
        planes = sobel_lib.sobel4x5_batched(srcs, dir_type=2)
        torch.cuda.synchronize()
        for i, (om, od) in enumerate(want):
            assert all(np.array_equal(o[i].cpu().numpy(), om) for o in outs)
            assert np.array_equal(planes[i][0].cpu().numpy(), om)
            assert np.array_equal(np.stack([d.cpu().numpy() for d in planes[i][1]]), od)
