"""The out-of-core Siddon forward's overlapped upload (pageable volumes from 80 MiB on whose 8-slice pieces fit the
pinned buffers): two and three slabs, each in at least three host pieces with a ragged last one, so that both pinned
buffers and the device stage are used again within a slab and from slab to slab; pinned volumes of the same sizes,
and 16-bit ones; against the resident projection, twice with the same buffers."""
import pytest
import torch

from _helpers import rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# host pieces are 16 MiB, in whole pieces of 8 slices: 16 slices of 512 x 500 in FP32, 32 in FP16; with slices of
# 700 x 690 a piece is 8 slices
@pytest.mark.parametrize("nvox,dt,n_slabs", [((512, 500, 101), torch.float32, 2), ((512, 500, 149), torch.float32, 3),
                                             ((512, 500, 203), torch.float16, 2), ((700, 690, 59), torch.float32, 2)])
@pytest.mark.parametrize("pinned", [False, True])
def test_overlapped_upload(nvox, dt, n_slabs, pinned):
    w = inputs.Workload("overlap", nvox, (256.0 / nvox[0],) * 3, (70, 66), (5.0, 5.0 * nvox[2] / nvox[0]), 6, 10, 3)
    x = torch.rand(nvox[::-1], generator=torch.Generator().manual_seed(3)).to(dt)
    assert x.numel() * x.element_size() >= 80 << 20
    h = x.pin_memory() if pinned else x
    plan = Plan(w.geometry_dict(), w.angles)
    slices = -(-nvox[2] // n_slabs)
    cap = (64 << 20) + 3 * 6 * 70 * 66 * 4 + (slices + 10) * nvox[0] * nvox[1] * x.element_size()
    assert plan.ooc_plan(0, "siddon", vol_dtype=dt, cap_bytes=cap)["n_slabs"] == n_slabs
    ref = plan.forward(x.to(DEV), "siddon", out_dtype=torch.float32).cpu().numpy()
    for _ in range(2):
        say(f"[overlapped upload] {nvox} {dt}, {n_slabs} slabs, pinned {pinned}")
        out = torch.zeros(plan.proj_shape)
        st = plan.forward_host(h, out, "siddon", cap_bytes=cap)
        assert st["n_slabs"] == n_slabs, st
        assert st["bytes_h2d"] >= x.numel() * x.element_size()
        assert rel_l2(out.numpy(), ref) <= 1e-6
        h = torch.flip(h, (0,))
        h = h.pin_memory() if pinned else h
        ref = plan.forward(h.to(DEV), "siddon", out_dtype=torch.float32).cpu().numpy()
