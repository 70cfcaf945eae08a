"""fp32 forward and adjoint on geometries of their column strips and row
ranges: strips that lie inside the image (one load a column pair), row ranges
of a few rows, rows that are only 4-byte aligned, and magnitudes of zero and
NaN beside ordinary ones.  Tolerances: those of test_gpu_f32."""
import numpy as np
import pytest

from test_gpu_f32 import check_bwd, check_fwd, f32_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def both(api, xt, gt, border):
    M = api.sobel4x5_f32_fwd(xt, border)
    dx = api.sobel4x5_f32_bwd(xt, gt, border)
    torch.cuda.synchronize()
    return M.cpu().numpy(), dx.cpu().numpy()


@pytest.mark.parametrize("border", [0, 1, 2, 3])
@pytest.mark.parametrize("h,w", [(5, 500), (8, 372), (9, 374), (13, 500), (17, 613), (41, 500), (90, 381)])
def test_inner_strips_and_short_ranges(oracle_mod, sobel_lib, gpu, border, h, w):
    x = f32_batch(2, h, w, 3 * h + w)
    ho, wo = sobel_lib.out_shape(h, w, border)
    g = np.random.default_rng(h + w).standard_normal((2, ho, wo)).astype(np.float32)
    # rows at odd multiples of 4 bytes
    xt = torch.zeros((2, h, w + 3), device=gpu)[:, :, 1:w + 1]
    gt = torch.zeros((2, ho, wo + 1), device=gpu)[:, :, 1:]
    xt.copy_(torch.from_numpy(x))
    gt.copy_(torch.from_numpy(g))
    M, dx = both(sobel_lib, xt, gt, border)
    check_fwd(oracle_mod, x, M, border)
    check_bwd(oracle_mod, x, g, dx, border)


def test_flat_patches_and_nan(oracle_mod, sobel_lib, gpu):
    """Rows that mix S = 0 with ordinary S give exact zeros and full accuracy;
    a NaN pixel reaches the outputs within its stencil and no others."""
    rng = np.random.default_rng(3)
    x = rng.random((1, 40, 500)).astype(np.float32)
    x[0, 10:30, 100:180] = np.float32(0.3)
    g = rng.standard_normal(x.shape).astype(np.float32)
    xt, gt = torch.from_numpy(x).to(gpu), torch.from_numpy(g).to(gpu)
    M, dx = both(sobel_lib, xt, gt, 0)
    check_fwd(oracle_mod, x, M, 0)
    check_bwd(oracle_mod, x, g, dx, 0)
    y = x.copy()
    y[0, 20, 300] = np.nan
    My, dy = both(sobel_lib, torch.from_numpy(y).to(gpu), gt, 0)
    inside = np.zeros(x.shape, bool)
    inside[0, 18:23, 298:303] = True
    assert np.isnan(My[inside]).any() and not np.isnan(My[~inside]).any()
    near = np.zeros(x.shape, bool)
    near[0, 16:25, 296:305] = True
    assert not np.isnan(dy[~near]).any() and np.array_equal(dy[~near], dx[~near])
