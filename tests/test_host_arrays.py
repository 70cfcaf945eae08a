"""The arrays that a pipe hands out: numpy arrays in every respect, whose memory
the pipe keeps for its next runs."""
import gc
import os

import numpy as np
import pytest

from paper_2305_00515_amd import synth

torch = pytest.importorskip("torch")


def check_ordinary(a):
    """Owns its data, can be resized in place, and a forked process reads it."""
    assert a.flags.owndata and a.flags.writeable and a.flags.c_contiguous and type(a) is np.ndarray
    assert not torch.cuda.is_available() or not torch.from_numpy(a).is_pinned()
    addr, inside = a.ctypes.data, False
    with open("/proc/self/smaps") as f:
        for line in f:
            w = line.split()
            if not w[0].endswith(":"):
                lo, hi = (int(x, 16) for x in w[0].split("-"))
                inside = lo <= addr < hi
            elif inside and w[0] == "VmFlags:":
                assert "dc" not in w and "io" not in w, line     # not inherited by a fork; device memory


def test_blocks_are_kept_and_bounded(sobel_lib):
    if sobel_lib._bind is None:
        pytest.skip("no binding built")
    pool = sobel_lib._Outputs()
    block = 1 << 19
    a = pool.array(500, 601)
    check_ordinary(a)
    a[:] = 7
    view, where = a[10:, 3:].T, a.ctypes.data
    del a
    b = pool.array(500, 601)
    assert b.ctypes.data != where and (view == 7).all() and pool._bytes == 2 * block
    del view
    a = pool.array(600, 500)
    assert a.ctypes.data == where and pool._bytes == 2 * block       # given back and taken again
    a[:] = 3
    a.resize((700, 1000))
    assert (a[:428].ravel()[:300000] == 3).all() and a.flags.owndata and pool._bytes == block
    pool.LIMIT = 2 * block
    some = [pool.array(500, 601) for _ in range(4)]
    assert pool._bytes == 2 * block and all(s.shape == (500, 601) for s in some)
    del some
    big = pool.array(1000, 1001)                                     # idle blocks make room
    assert pool._bytes <= 2 * block
    assert pool.array(10, 10).shape == (10, 10) and pool.array(0, 7).shape == (0, 7)
    assert pool.array(-4, -1000000).shape == (0, 0)
    with pytest.raises((MemoryError, ValueError)):
        pool.array(1 << 40, 1 << 10)
    pool.close()
    assert pool._bytes == block                                      # b
    kept = pool.array(500, 601)
    del b, pool
    gc.collect()
    kept[:], big[:] = 1, 2
    assert kept.sum() == 300500 and big.sum() == 2002000


def test_numpy_is_as_before_outside(sobel_lib):
    if sobel_lib._bind is None:
        pytest.skip("no binding built")
    pool = sobel_lib._Outputs()
    a = pool.array(500, 601)
    b = np.empty((500, 601), np.uint8)
    copy = a.copy()
    assert pool._bytes == 1 << 19 and b.flags.owndata and copy.flags.owndata


def test_a_forked_process_reads_them(sobel_lib):
    pool = sobel_lib._Outputs()
    a = pool.array(500, 601)
    a[:] = 9
    pid = os.fork()
    if pid == 0:
        os._exit(0 if (a == 9).all() else 1)
    assert os.waitpid(pid, 0)[1] == 0


@pytest.mark.gpu
def test_pipe_outputs_are_ordinary_arrays(oracle_mod, sobel_lib, gpu):
    imgs = [synth.rect_image(700, 901, 5), synth.rect_image(64, 64, 6)]
    pipe = sobel_lib.Pipe(901, 700)
    want = [oracle_mod.sobel_u8(m, want_dir=False)[0] for m in imgs]
    for _ in range(3):
        outs = pipe.run(imgs)
        for o, w in zip(outs, want):
            check_ordinary(o)
            assert np.array_equal(o, w)
    kept = outs[0]
    pipe.run([imgs[0][:, ::-1].copy()])
    assert np.array_equal(kept, want[0])
    pipe.close()
    kept.resize((701, 901), refcheck=False)
    assert np.array_equal(kept[:700], want[0])
