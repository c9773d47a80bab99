"""The exact adjoint's column kernel with two neighbouring voxels per lane, against the CPU FP64 oracle: slice
counts around its groups of 128 (one lane's pair cut off), 2 to 4 rows that can meet a pair (and more, where
voxels are taken one by one), the source plane between the voxels of a pair, through one, and on a row of the
detector, angle ranges and accumulation, vertical views, and the column-major slabs of the out-of-core form."""
import numpy as np
import pytest
import torch

from _helpers import TOL_BP, rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# slices, slice height, rows, row pitch, volume z offset
CASES = [(2, 1.0, 40, 1.6, 0.0), (65, 1.0, 71, 1.6, 0.0), (66, 1.0, 70, 1.6, 0.5), (127, 0.8, 91, 1.6, 0.0),
         (128, 0.8, 90, 1.6, 0.4), (129, 0.8, 91, 1.6, 0.3), (130, 0.8, 64, 2.9, -0.2), (200, 0.5, 99, 1.1, 0.0),
         (257, 0.4, 120, 1.1, 7.0), (390, 0.3, 101, 1.3, 0.15), (520, 0.2, 101, 1.3, 0.0), (90, 1.0, 140, 1.0, 0.5),
         (90, 1.0, 260, 0.5, 0.0)]


def _work(nz, dz, nv, dv, oz):
    return inputs.Workload("adj_pairs", (15, 14, nz), (1.4, 1.5, dz), (27, nv), (1.3, dv), 11, 10, 3,
                           off_origin=(2.0, -1.0, oz), off_detector=(0.31, 0.0))


@pytest.mark.parametrize("case", CASES)
def test_adjoint_pairs_match_the_oracle(orc, case):
    w = _work(*case)
    y = inputs.random_array((11, w.ndet[1], w.ndet[0]), 5, kind="uniform")
    say(f"[adjoint pairs] {case}")
    og = orc.Geometry.from_dict(w.geometry_dict())
    yd = torch.from_numpy(y).to(DEV)
    for scan in (w.angles + 0.1, inputs.helical_views(w.DSO, w.DSD, w.angles + 0.1, pitch=13.0, z0=-6.0)):
        plan = Plan(w.geometry_dict(), scan)
        ref = orc.siddon_adj(og, scan, y.astype(np.float64))
        assert rel_l2(plan.backproject(yd, "adjoint").cpu().numpy(), ref) <= TOL_BP
        out = plan.backproject(yd[:4].contiguous(), "adjoint", angle_begin=0, angle_end=4)
        plan.backproject(yd[4:].contiguous(), "adjoint", out=out, accumulate=True, angle_begin=4, angle_end=11)
        assert rel_l2(out.cpu().numpy(), ref) <= TOL_BP


@pytest.mark.parametrize("slices", [129, 60, 33])
def test_adjoint_pairs_slabs(slices):
    w = _work(129, 0.8, 91, 1.6, 0.3)
    y = inputs.random_array((11, 91, 27), 6, kind="uniform")
    plan = Plan(w.geometry_dict(), w.angles)
    out = torch.zeros(plan.vol_shape)
    cap = (64 << 20) + 11 * (2 * 91 + 2 * 93) * 27 * 4 + (slices + 8) * 15 * 14 * 4
    say(f"[adjoint pairs] slabs of about {slices}")
    plan.backproject_host(torch.from_numpy(y), out, "adjoint", cap_bytes=cap)
    ref = plan.backproject(torch.from_numpy(y).to(DEV), "adjoint").cpu()
    assert rel_l2(out.numpy(), ref.numpy()) <= 1e-5
