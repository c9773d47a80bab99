"""The out-of-core Siddon forward's upload of pageable and pinned volumes: slabs of less than one piece, of
several pieces with a ragged last one, and slices so large that a piece passes through the pinned buffers in
parts, against the resident projection."""
import pytest
import torch

from _helpers import rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nvox,slices", [((64, 48, 20), 20), ((64, 48, 21), 6), ((512, 500, 45), 19), ((1500, 1490, 11), 9)])
@pytest.mark.parametrize("pinned", [False, True])
def test_upload_pieces(nvox, slices, pinned):
    w = inputs.Workload("upload", nvox, (256.0 / nvox[0],) * 3, (70, 66), (5.0, 5.0 * nvox[2] / nvox[0]), 6, 10, 3)
    x = torch.rand(nvox[::-1], generator=torch.Generator().manual_seed(3))
    h = x.pin_memory() if pinned else x
    plan = Plan(w.geometry_dict(), w.angles)
    # the reserve, three chunks of all angles, the slab with its pads and the 8-slice stage
    cap = (64 << 20) + 3 * 6 * 70 * 66 * 4 + (slices + 10) * nvox[0] * nvox[1] * 4
    say(f"[upload] {nvox}, slabs of {slices}, pinned {pinned}")
    out = torch.zeros(plan.proj_shape)
    st = plan.forward_host(h, out, "siddon", cap_bytes=cap)
    assert nvox[0] < 512 or st["n_slabs"] > 1, st   # (small volumes: the planner shrinks the chunks instead)
    assert rel_l2(out.numpy(), plan.forward(x.to(DEV), "siddon").cpu().numpy()) <= 1e-6
