"""The column Siddon walk that takes two neighbouring rows per lane, against the CPU FP64 oracle: odd and
even row counts around a wave's 128 rows, rows less than one slot apart everywhere, more than one, a change
between the two inside the grid (and beyond two, where the walk with rows 64 apart stays), detectors wholly
above or below the source, grids that the rows leave at both ends, single slices, 16-bit storage, views, and
a voxel that is not finite (it reaches only the rays that come within a slice of it)."""
import numpy as np
import pytest
import torch

from _helpers import TOL_PROJ, rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# rows, row pitch (mm): with 1 mm slices the rows lie 0.56 .. 0.78 of the pitch apart in the grid
CASES = [(65, 1.1, 0.0), (66, 1.1, 0.3), (127, 1.6, 0.0), (128, 1.6, 0.4), (129, 1.6, -0.2), (130, 2.2, 0.0),
         (257, 0.7, 0.1), (90, 2.9, 0.0), (70, 1.6, 90.0), (70, 1.6, -90.0), (200, 2.4, 20.0), (75, 1.5, 0.0)]


def _work(nv, dv, offv, nz=40):
    return inputs.Workload("pairs", (41, 38, nz), (1.0, 1.1, 1.0), (33, nv), (2.1, dv), 17, 10, 3,
                           off_origin=(2.0, -1.0, 0.7), off_detector=(0.31, offv))


@pytest.mark.parametrize("nv,dv,offv", CASES)
def test_pairs_match_the_oracle(orc, nv, dv, offv):
    w = _work(nv, dv, offv)
    vol = np.random.default_rng(5).uniform(0, 1, w.nvox[::-1]).astype(np.float32)
    say(f"[siddon pairs] {nv} rows of {dv} mm, offset {offv}")
    ref = orc.siddon_fwd(orc.Geometry.from_dict(w.geometry_dict()), w.angles, vol.astype(np.float64))
    plan = Plan(w.geometry_dict(), w.angles)
    x = torch.from_numpy(vol).to(DEV)
    assert rel_l2(plan.forward(x, "siddon").cpu().numpy(), ref) <= TOL_PROJ
    # accumulation, and an angle range that starts inside a group of angles
    out = plan.forward(x, "siddon", angle_begin=3, angle_end=11)
    plan.forward(x, "siddon", out=out, accumulate=True, angle_begin=3, angle_end=11)
    assert rel_l2(out.cpu().numpy(), 2.0 * ref[3:11]) <= TOL_PROJ
    h = x.half()   # 16-bit storage: the same walk of the same values
    assert rel_l2(plan.forward(h, "siddon", out_dtype=torch.float32).cpu().numpy(),
                  plan.forward(h.float(), "siddon").cpu().numpy()) <= 1e-6


@pytest.mark.parametrize("nz", [1, 2, 3])
def test_pairs_thin_grids_and_views(orc, nz):
    w = _work(75, 1.5, 0.0, nz)
    vol = np.random.default_rng(6).uniform(0, 1, w.nvox[::-1]).astype(np.float32)
    og = orc.Geometry.from_dict(w.geometry_dict())
    x = torch.from_numpy(vol).to(DEV)
    for scan in (w.angles, inputs.helical_views(w.DSO, w.DSD, w.angles, pitch=12.0, z0=-6.0)):
        say(f"[siddon pairs] {nz} slices, {np.ndim(scan)}-d scan")
        got = Plan(w.geometry_dict(), scan).forward(x, "siddon").cpu().numpy()
        assert rel_l2(got, orc.siddon_fwd(og, scan, vol.astype(np.float64))) <= TOL_PROJ


# (rows outside the grid are held at its first or last slice with weight zero, so those two slices are left out)
@pytest.mark.parametrize("at", [(1, 0, 0), (20, 19, 20), (38, 37, 40), (1, 37, 40), (38, 0, 0)])
@pytest.mark.parametrize("dv", [1.1, 1.6, 2.4])
def test_pairs_non_finite_voxel(orc, at, dv):
    w = _work(129, dv, 0.0)
    vol = np.random.default_rng(7).uniform(0, 1, w.nvox[::-1]).astype(np.float32)
    near = np.zeros(w.nvox[::-1])
    near[max(at[0] - 1, 0):at[0] + 2, at[1], at[2]] = 1.0
    reach = orc.siddon_fwd(orc.Geometry.from_dict(w.geometry_dict()), w.angles, near) > 0
    through = np.zeros_like(near)
    through[at] = 1.0
    hit = orc.siddon_fwd(orc.Geometry.from_dict(w.geometry_dict()), w.angles, through) > 1e-3
    vol[at] = np.nan
    p = Plan(w.geometry_dict(), w.angles).forward(torch.from_numpy(vol).to(DEV), "siddon").cpu().numpy()
    assert np.all(np.isnan(p[hit])) and not np.any(np.isnan(p[~reach]))
