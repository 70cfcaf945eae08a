"""Batches with directional planes: the plane type chooses the pixels a lane
holds, and images of one batch may ask for different outputs."""
import ctypes

import numpy as np
import pytest

from paper_2305_00515_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (3, 3), (2, 65), (9, 4), (40, 64), (33, 61), (5, 4099), (130, 5), (64, 320)]
DTYPE = {1: torch.int16, 2: torch.int32}


def test_int32_planes_take_four_pixels_a_lane(sobel_lib, gpu):
    """One store of 16 bytes a lane and plane."""
    srcs = [torch.zeros((40, 64), dtype=torch.uint8, device=gpu)]
    for dt, ppl in ((1, 8), (2, 4)):
        mags = [torch.empty_like(srcs[0])]
        dirs = [[torch.empty((40, 64), dtype=DTYPE[dt], device=gpu) for _ in range(4)]]
        plan = sobel_lib.Plan(srcs, mags, dir_type=dt, dirs=dirs)
        assert plan.info()["px_per_lane"] == ppl
        plan.close()


@pytest.mark.parametrize("types", [(2,), (2, 0), (1, 2), (1, 2, 0), (0, 2, 1)])
@pytest.mark.parametrize("queue", ["0", "1"])
@pytest.mark.parametrize("pad", [0, 3])
def test_mixed_outputs(oracle_mod, sobel_lib, gpu, monkeypatch, types, queue, pad):
    """int32 planes alone, beside images with none, and beside int16 ones; some
    without a magnitude; rows of whole lines and others; both grid forms."""
    api = sobel_lib
    monkeypatch.setenv("SOBEL4X5_BATCH_STATIC", queue)
    for border in (0, 2, 3):
        imgs = [synth.rect_image(h, w, 7 * h + w) % 6 for h, w in SIZES]
        srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
        arr, outs, keep = (api.Image * len(imgs))(), (api.Outputs * len(imgs))(), []
        for i, s in enumerate(srcs):
            h, w = s.shape
            t = types[i % len(types)]
            pitch = (w + 63) // 64 * 64 + pad
            mag = torch.full((h, pitch), 9, dtype=torch.uint8, device=gpu) if t == 0 or i % 3 else None
            dirs = [torch.full((h, pitch), 9, dtype=DTYPE[t], device=gpu) for _ in range(4)] if t else []
            keep.append((mag, dirs))
            arr[i].src, arr[i].height, arr[i].width, arr[i].src_pitch = s.data_ptr(), h, w, s.stride(0)
            if mag is not None:
                outs[i].mag, outs[i].mag_pitch = mag.data_ptr(), pitch
            outs[i].dir_type = t
            for k, d in enumerate(dirs):
                outs[i].dir[k] = d.data_ptr()
                outs[i].dir_pitch = pitch * d.element_size()
        h = ctypes.c_void_p()
        assert api.lib.sobel4x5_plan_create_ex(arr, outs, len(imgs), border, 0, ctypes.byref(h)) == 0
        assert api.lib.sobel4x5_plan_launch(h, None) == 0
        torch.cuda.synchronize()
        assert api.lib.sobel4x5_plan_destroy(h) == 0
        for m, (mag, dirs) in zip(imgs, keep):
            w = m.shape[1]
            om, od = oracle_mod.sobel_u8(m, border)
            for got, want in zip(([mag] if mag is not None else []) + dirs,
                                 ([om] if mag is not None else []) + list(od)):
                got = got.cpu().numpy()
                assert np.array_equal(got[:, :w], want), (m.shape, border)
                assert (got[:, w:] == 9).all(), (m.shape, border)
