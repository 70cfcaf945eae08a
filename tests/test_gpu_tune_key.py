"""What a tuned shape is filed under: everything that selects the kernel and the
shape that tuning starts from."""
import pytest

from paper_2305_00515_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_tuned_shapes_of_other_outputs_are_not_reused(sobel_lib, gpu, tmp_path, monkeypatch):
    """The same images with rows of whole lines and with rows that share them,
    with int16 and with int32 planes, with planes alone: five entries, and each
    again is served from its own."""
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("SOBEL4X5_TUNE_CACHE", str(path))
    srcs = [torch.from_numpy(synth.rect_image(48, 128, i)).to(gpu) for i in range(3)]

    def plan(dtype=None, pad=0, mag=True):
        new = lambda t: [torch.empty((48, 128 + pad), dtype=t, device=gpu)[:, :128] for _ in srcs]
        mags = new(torch.uint8) if mag else [None] * 3
        if dtype is None:
            return sobel_lib.Plan(srcs, mags, autotune=True)
        planes = [new(dtype) for _ in range(4)]
        return sobel_lib.Plan(srcs, mags, autotune=True, dir_type=1 if dtype == torch.int16 else 2,
                              dirs=[[p[i] for p in planes] for i in range(3)])

    forms = [dict(), dict(pad=1), dict(dtype=torch.int16), dict(dtype=torch.int32), dict(dtype=torch.int16, mag=False)]
    for _ in range(2):
        for f in forms:
            plan(**f).close()
        keys = [line.split()[0] for line in path.read_text().splitlines()]
        assert len(keys) == len(set(keys)) == len(forms)
