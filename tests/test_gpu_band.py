"""GPU parity of the banded matrix-core kernels (u8_band.hpp) against the CPU
oracle, bit-exact, where their loads and tiles can go wrong."""
import numpy as np
import pytest

from paper_2305_00515_amd import synth
from test_gpu_u8 import run

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def check_mag(oracle_mod, api, img, dev, border, **kw):
    mag, _, flat = run(api, img, dev, border, 0, **kw)
    om, _ = oracle_mod.sobel_u8(np.ascontiguousarray(img), border, want_dir=False)
    bad = int((mag != om).sum())
    assert bad == 0, "border %d, %s, %s: %d pixels differ" % (border, img.shape, kw, bad)


# 16-column tiles, quads of 4 rows, waves of 16 tiles (256 columns), rows of
# fewer than 4 bytes: widths and heights on both sides of each
WIDTHS = [1, 2, 3, 4, 5, 7, 15, 16, 17, 19, 20, 23, 24, 31, 33, 40, 127, 240, 255, 257, 272, 529]


@pytest.mark.parametrize("border", [0, 1, 2, 3])
@pytest.mark.parametrize("w", WIDTHS)
def test_widths_heights_and_borders(oracle_mod, sobel_lib, gpu, border, w):
    for h in (1, 2, 3, 4, 5, 8, 9, 13, 34):
        if border == 1 and (h < 5 or w < 5):
            continue
        # small values: the magnitudes do not saturate
        check_mag(oracle_mod, sobel_lib, synth.rect_image(h, w, 97 * h + w) % 5, gpu, border)


@pytest.mark.parametrize("offset", [0, 1, 2, 3, 4, 9])
def test_any_alignment(oracle_mod, sobel_lib, gpu, offset):
    """Rows at every byte alignment, in and out, wide enough for waves whose
    windows all lie inside the image."""
    img = synth.rect_image(53, 1100, 40 + offset) % 7
    for pitch in (1100, 1101, 1102, 1103, 1280):
        for border in (0, 1):
            check_mag(oracle_mod, sobel_lib, img, gpu, border, pitch=pitch, offset=offset, mag_pitch=1100 + offset)


@pytest.mark.parametrize("h,w", [(520, 2050), (1031, 4001), (4099, 2057), (70000, 33)])
def test_bands_of_several_steps(oracle_mod, sobel_lib, gpu, h, w):
    """Bands of 2 to 8 steps, even and odd last bands, tile rows that end
    inside a wave, more waves than one round."""
    img = synth.rect_image(h, w, h + w)
    for border in (0, 3):
        check_mag(oracle_mod, sobel_lib, img, gpu, border)


# planes: tiles of 8 columns (int16) or 4 (int32), stores of 16 bytes a plane
@pytest.mark.parametrize("op", [0, 1, 2])
@pytest.mark.parametrize("dir_type", [1, 2])
@pytest.mark.parametrize("w", [3, 4, 5, 7, 8, 9, 12, 17, 64, 65, 129, 270])
def test_planes(oracle_mod, sobel_lib, gpu, op, dir_type, w):
    """Planes of every operator, with and without the magnitude, rows at odd
    element offsets, guard columns untouched."""
    dt = torch.int16 if dir_type == 1 else torch.int32
    r = 1 if op == 2 else 2
    for h in (3, 5, 9, 22):
        img = synth.rect_image(h, w, 31 * h + w) % 9
        src = torch.from_numpy(img).to(gpu)
        for border in (0, 1, 2, 3):
            ho, wo = (h - 2 * r, w - 2 * r) if border == 1 else (h, w)
            if ho < 1 or wo < 1:
                continue
            for want_mag in (True, False):
                base = [torch.full((ho, wo + 3), 77, dtype=dt, device=gpu) for _ in range(4 if op == 0 else 2)]
                mag, _ = sobel_lib.sobel4x5_u8_op(src, op, border, want_mag=want_mag, dir_type=dir_type,
                                                  dirs=[b[:, 1:wo + 1] for b in base])
                if op == 0:
                    om, od = oracle_mod.sobel_u8(img, border)
                else:
                    om, od = oracle_mod.sobel_u8_2dir(img, 5 if op == 1 else 3, border)
                torch.cuda.synchronize()
                got = np.stack([b.cpu().numpy() for b in base])
                what = "op %d, border %d, %dx%d" % (op, border, h, w)
                assert np.array_equal(got[:, :, 1:wo + 1], od), what
                assert (got[:, :, 0] == 77).all() and (got[:, :, wo + 1:] == 77).all(), what
                if want_mag:
                    assert np.array_equal(mag.cpu().numpy(), om), what


def antisymmetric(rng, amp, nonzero):
    """Four kernels of `nonzero` random pairs of weights up to amp."""
    w = np.zeros((4, 5, 5), np.int64)
    taps = [(i, j) for i in range(3) for j in range(5) if (i, j) < (2, 2)]
    for k in range(4):
        for t in rng.choice(12, nonzero, replace=False):
            i, j = taps[t]
            w[k, i, j] = rng.integers(-amp, amp + 1)
            w[k, 4 - i, 4 - j] = -w[k, i, j]
    return w.astype(np.int32)


# sums of |weights| below and above 181 (squares with and without the clamp),
# and up to 128 for int16 planes
@pytest.mark.parametrize("amp,nonzero,dir_type", [(7, 12, 2), (127, 12, 2), (127, 1, 2), (5, 12, 1), (64, 1, 1)])
def test_weighted_planes(oracle_mod, sobel_lib, gpu, amp, nonzero, dir_type):
    rng = np.random.default_rng(amp + nonzero)
    w = antisymmetric(rng, amp, nonzero)
    for h, wd in [(3, 2), (9, 17), (33, 70), (21, 300)]:
        img = synth.rect_image(h, wd, h + wd)
        for im in (img, img % 3):
            src = torch.from_numpy(im).to(gpu)
            for border in (0, 1, 2, 3):
                if border == 1 and min(h, wd) < 5:
                    continue
                mag, dirs = sobel_lib.sobel4x5_u8_weighted(src, w, border, dir_type=dir_type)
                om, od = oracle_mod.sobel_u8(im, border, weights=w)
                torch.cuda.synchronize()
                assert np.array_equal(mag.cpu().numpy(), om), (h, wd, border)
                assert np.array_equal(np.stack([d.cpu().numpy() for d in dirs]), od), (h, wd, border)


@pytest.mark.parametrize("sizes,planes", [
    ([(1, 1), (3, 2), (2, 300), (64, 15), (17, 16), (33, 257), (5, 4099), (1030, 31)], 0),
    ([(40, 64), (64, 128), (16, 32)], 1),           # rows of whole 64-byte pieces: stores past the L2
    ([(40, 64), (9, 33), (31, 7), (2, 2)], 1),      # other rows
    ([(40, 64), (9, 33), (31, 7), (2, 2)], 2),
])
def test_batches(oracle_mod, sobel_lib, gpu, sizes, planes):
    """Wave-tiles that end inside a row of tiles, narrow images, both kinds of
    plane stores; plan, one-shot and allocation-free call."""
    imgs = [synth.rect_image(h, w, 7 * h + w) % 6 for h, w in sizes]
    srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
    dt = {1: torch.int16, 2: torch.int32}.get(planes)
    for border in (0, 2, 3):
        want = [oracle_mod.sobel_u8(m, border) for m in imgs]
        mags = [torch.full(m.shape, 9, dtype=torch.uint8, device=gpu) for m in imgs]
        dirs = [[torch.full(m.shape, 9, dtype=dt, device=gpu) for _ in range(4)] for m in imgs] if planes else None
        plan = sobel_lib.Plan(srcs, mags, border, dir_type=planes, dirs=dirs)
        plan.launch()
        shot = sobel_lib.sobel4x5_batched(srcs, border=border, dir_type=planes)
        got = [[m] + (list(dirs[i]) if planes else []) for i, m in enumerate(mags)]
        more = [[r[0]] + list(r[1]) for r in shot] if planes else [[r] for r in shot]
        if not planes:
            more = [a + b for a, b in zip(more, [[r] for r in sobel_lib.sobel4x5_batched_noalloc(srcs, border=border)])]
        torch.cuda.synchronize()
        for i, (om, od) in enumerate(want):
            for k, t in enumerate(got[i] + more[i]):
                plane = (k % 5) if planes else 0
                ref = om if plane == 0 else od[plane - 1]
                assert np.array_equal(t.cpu().numpy(), ref), (sizes[i], border, k)
        plan.close()


@pytest.mark.parametrize("count", [1, 2, 47, 48, 49, 63])
def test_one_shot_batches_of_any_count(oracle_mod, sobel_lib, gpu, count):
    """Up to 48 images travel in the kernel's arguments, more through a plan:
    the same results on both sides of the line, call after call with other
    buffers, also captured into a graph (up to 48)."""
    rng = np.random.default_rng(count)
    sizes = [(int(h), int(w)) for h, w in rng.integers(1, 90, (count, 2))]
    for rep in range(2):
        imgs = [synth.rect_image(h, w, 100 * rep + h + w) % 6 for h, w in sizes]
        srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
        border = 3 * rep
        mags = sobel_lib.sobel4x5_batched(srcs, border=border)
        torch.cuda.synchronize()
        for m, t in zip(imgs, mags):
            assert np.array_equal(t.cpu().numpy(), oracle_mod.sobel_u8(m, border, want_dir=False)[0]), m.shape
    if count <= 48:
        out = [torch.empty_like(s) for s in srcs]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            sobel_lib.sobel4x5_batched(srcs, out, border=border)
        for _ in range(3):
            for t in out:
                t.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(out, mags))


def test_plan_launches_under_capture(oracle_mod, sobel_lib, gpu):
    """A plan launches its kernel as such, so its launches can be captured."""
    imgs = [synth.rect_image(h, w, h + w) for h, w in ((5, 9), (64, 300), (131, 77))]
    srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
    mags = [torch.empty_like(s) for s in srcs]
    plan = sobel_lib.Plan(srcs, mags)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.launch()
    for _ in range(3):
        for t in mags:
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        for m, t in zip(imgs, mags):
            assert np.array_equal(t.cpu().numpy(), oracle_mod.sobel_u8(m, 0, want_dir=False)[0]), m.shape
