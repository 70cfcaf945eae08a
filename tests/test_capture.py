"""Calls whose stream is being captured into a graph.  On the CPU: the C-ABI
layer against a recorded stand-in for the runtime and the kernels
(tests/sanitize/capture_driver.cpp), under the host sanitizers.  On the GPU: the
same rules through the library."""
import os
import subprocess

import numpy as np
import pytest

from paper_2305_00515_amd import synth
from test_sanitizers import CLANGXX, ROOT, SAN, SANFLAGS

torch = pytest.importorskip("torch")


@pytest.mark.skipif(not os.path.exists(CLANGXX), reason="clang from ROCm not found")
def test_captured_calls_on_the_host(tmp_path):
    exe = str(tmp_path / "capture_driver")
    subprocess.run([CLANGXX, "-std=c++17", "-w"] + SANFLAGS +
                   ["-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    os.path.join(ROOT, "paper_2305_00515_amd", "csrc", "sobel4x5_api.cpp"),
                    os.path.join(SAN, "capture_driver.cpp"), "-L/opt/rocm/lib", "-Wl,-rpath,/opt/rocm/lib",
                    "-lamdhip64", "-o", exe], check=True)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0", UBSAN_OPTIONS="halt_on_error=1")
    r = subprocess.run([exe], capture_output=True, text=True, env=env)
    assert r.returncode == 0 and "capture checks ok" in r.stdout, r.stdout + r.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("planes", [False, True])
def test_batches_of_a_cached_plan_are_refused_under_capture(oracle_mod, sobel_lib, gpu, planes):
    """More than 48 images, or planes: refused while capturing, also when the
    plan is cached already; the capture goes on, and the call works after it."""
    imgs = [synth.rect_image(20 + i, 33, i) % 6 for i in range(3 if planes else 49)]
    srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
    mags = [torch.empty_like(s) for s in srcs]
    dirs = [[torch.empty(s.shape, dtype=torch.int16, device=gpu) for _ in range(4)] for s in srcs] if planes else None
    call = lambda: sobel_lib.sobel4x5_batched(srcs, mags, dir_type=1 if planes else 0, dirs=dirs)
    one = torch.zeros_like(srcs[0])
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        with pytest.raises(sobel_lib.SobelError) as e:
            call()
        assert e.value.code == sobel_lib.EUNSUPPORTED and "plan" in str(e.value)
        sobel_lib.sobel4x5_u8(srcs[0], mag=one)
    for t in mags:
        t.zero_()
    g.replay()
    with torch.cuda.stream(stream):
        call()
    torch.cuda.synchronize()
    want = [oracle_mod.sobel_u8(m, want_dir=False)[0] for m in imgs]
    assert np.array_equal(one.cpu().numpy(), want[0])
    assert all(np.array_equal(t.cpu().numpy(), w) for t, w in zip(mags, want))


@pytest.mark.gpu
@pytest.mark.parametrize("count", [3, 49, 100])
def test_captured_noalloc_call_is_its_own(oracle_mod, sobel_lib, gpu, count):
    """Batch A captured through the allocation-free call, batch B run eagerly
    through it, A replayed: A's outputs, call after call."""
    def batch(n, seed):
        imgs = [synth.rect_image(17 + (7 * i + seed) % 40, 21 + (11 * i) % 60, seed + i) % 6 for i in range(n)]
        srcs = [torch.from_numpy(m).to(gpu) for m in imgs]
        return imgs, srcs, [torch.zeros_like(s) for s in srcs]
    a, b = batch(count, 1), batch(count + 5, 500)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        sobel_lib.sobel4x5_batched_noalloc(a[1], a[2])
    for _ in range(3):
        for t in a[2] + b[2]:
            t.zero_()
        sobel_lib.sobel4x5_batched_noalloc(b[1], b[2])
        g.replay()
        torch.cuda.synchronize()
        for imgs, _, mags in (a, b):
            for m, t in zip(imgs, mags):
                assert np.array_equal(t.cpu().numpy(), oracle_mod.sobel_u8(m, want_dir=False)[0]), m.shape
