"""TV steps at the edges of the two-pass kernels' tiles (64 columns x 8 rows, runs of 4 to 32 slices): odd
and even step counts (the steps alternate between two arrays), FP32 and 16-bit images, an eps below the
smallest normal number, images that are not finite (left unchanged), against the FP64 oracle."""
import numpy as np
import pytest
import torch

from _helpers import rel_l2, say
from paper_1905_03748_amd.operators import tv_steps

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _geo(shape):
    return dict(DSO=1000.0, DSD=1500.0, nVoxel=shape[::-1], dVoxel=(1.0, 1.0, 1.0), offOrigin=(0, 0, 0),
                nDetector=(8, 8), dDetector=(1.0, 1.0), offDetector=(0, 0), accuracy=0.5)


@pytest.mark.parametrize("shape", [(1, 1, 1), (1, 9, 65), (4, 8, 64), (5, 7, 63), (33, 17, 129), (65, 130, 260)])
@pytest.mark.parametrize("nsteps", [1, 2, 3])
def test_tv_tile_edges(orc, shape, nsteps):
    x0 = np.random.default_rng(91).uniform(0, 1, shape).astype(np.float32)
    say(f"[tv passes] {shape}, {nsteps} steps")
    x = torch.from_numpy(x0).to(DEV)
    assert tv_steps(_geo(shape), x, nsteps, 0.01).data_ptr() == x.data_ptr()
    # FP32 steps: each rounds x once (6e-8) and moves it by 1 % along a direction good to a few ulps
    assert rel_l2(x.cpu().numpy(), orc.tv_steps(x0.astype(np.float64), nsteps, 0.01)) <= 1e-6
    h = torch.from_numpy(x0).to(DEV).half()
    f = h.float()
    tv_steps(_geo(shape), h, nsteps, 0.01)
    tv_steps(_geo(shape), f, nsteps, 0.01)
    assert torch.equal(h, f.half())


def test_tv_tiny_eps_and_non_finite(orc):
    shape = (9, 10, 70)
    x0 = np.random.default_rng(92).uniform(0, 1, shape).astype(np.float32)
    x0[:, :5] = 0.25   # a flat part: the square root of eps alone
    x = torch.from_numpy(x0).to(DEV)
    tv_steps(_geo(shape), x, 2, 0.01, eps=1e-39)
    ref = torch.from_numpy(x0).to(DEV)
    tv_steps(_geo(shape), ref, 2, 0.01, eps=1e-30)
    assert torch.isfinite(x).all() and rel_l2(x.cpu().numpy(), ref.cpu().numpy()) <= 1e-6
    for bad in (float("inf"), float("nan")):
        y0 = torch.from_numpy(x0).to(DEV)
        y0[3, 4, 5] = bad
        y = y0.clone()
        tv_steps(_geo(shape), y, 3, 0.01)
        assert torch.equal(y.view(torch.int32), y0.view(torch.int32))
