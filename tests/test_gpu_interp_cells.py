"""The interpolated projector's 32-bit cell offsets against the CPU FP64 oracle: grids of one and two voxels
along an axis, rows and columns that miss the grid or graze its faces, every storage type, tilted detectors
(several samples per trip), and a voxel that is not finite (no ray that stays three voxels away sees it)."""
import numpy as np
import pytest
import torch

from _helpers import TOL_PROJ, rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _work(nvox, ndet):
    return inputs.Workload("cells", nvox, (1.0, 1.2, 0.9), ndet, (2.3, 2.1), 13, 10, 3, off_origin=(1.0, -2.0, 0.4),
                           off_detector=(0.4, -0.3))


@pytest.mark.parametrize("nvox", [(1, 1, 1), (2, 31, 1), (33, 1, 30), (37, 30, 2), (41, 38, 35)])
@pytest.mark.parametrize("ndet", [(7, 5), (33, 70), (40, 131)])
@pytest.mark.parametrize("scan", ["circle", "helix", "carm"])
def test_cells_match_the_oracle(orc, nvox, ndet, scan):
    w = _work(nvox, ndet)
    views = {"circle": w.angles, "helix": inputs.helical_views(w.DSO, w.DSD, w.angles, pitch=12.0, z0=-6.0),
             "carm": inputs.carm_views(w.DSO, w.DSD, w.angles, 5, tilt_deg=12.0, jitter_mm=4.0, orbit_tilt_deg=6.0)}[scan]
    vol = np.random.default_rng(5).uniform(0, 1, nvox[::-1]).astype(np.float32)
    say(f"[interp cells] {nvox} {ndet} {scan}")
    plan = Plan(w.geometry_dict(), views)
    x = torch.from_numpy(vol).to(DEV)
    ref = orc.interp_fwd(orc.Geometry.from_dict(w.geometry_dict()), views, vol.astype(np.float64))
    assert rel_l2(plan.forward(x, "interp").cpu().numpy(), ref) <= TOL_PROJ
    for dt in (torch.float16, torch.bfloat16):
        h = x.to(dt)
        assert torch.equal(plan.forward(h, "interp", out_dtype=torch.float32), plan.forward(h.float(), "interp"))


@pytest.mark.parametrize("at", [(0, 0, 0), (17, 19, 20), (34, 37, 40)])
def test_cells_non_finite_voxel(orc, at):
    w = _work((41, 38, 35), (40, 131))
    vol = np.random.default_rng(7).uniform(0, 1, (35, 38, 41)).astype(np.float32)
    near = np.zeros((35, 38, 41))
    near[tuple(slice(max(a - 3, 0), a + 4) for a in at)] = 1.0
    reach = orc.interp_fwd(orc.Geometry.from_dict(w.geometry_dict()), w.angles, near) > 0
    vol[at] = np.nan
    p = Plan(w.geometry_dict(), w.angles).forward(torch.from_numpy(vol).to(DEV), "interp").cpu().numpy()
    assert np.any(np.isnan(p)) and not np.any(np.isnan(p[~reach]))
