"""The staged voxel backprojections (FDK and pseudo-matched) where a tile's detector window is copied
straight into LDS (it lies on the detector) and where it is not, against the CPU FP64 oracle: detectors
narrower than, as wide as and wider than a window's LDS row (37 pixels), windows that need more than one
round of copies, rows that climb by less and by more than one per voxel, ragged grids, 16-bit storage.
"""
import numpy as np
import pytest
import torch

from _helpers import TOL_BP, rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kind", ["fdk", "pm"])
@pytest.mark.parametrize("ndet,ddet", [((36, 40), (2.6, 2.4)), ((37, 61), (2.6, 1.1)), ((38, 90), (2.6, 0.9)),
                                       ((91, 75), (1.25, 1.3)), ((120, 33), (0.9, 3.1)), ((64, 200), (2.0, 0.5))])
def test_staged_windows(orc, kind, ndet, ddet):
    # (64, 200): windows of about 70 rows, more than the four copies whose offsets are formed once
    w = inputs.Workload("staging", (37, 34, 35), (1.7, 1.8, 1.6), ndet, ddet, 19, 10, 5, off_origin=(1.1, -0.6, 0.8),
                        off_detector=(0.4, -0.3))
    y = inputs.random_array((19, ndet[1], ndet[0]), 77, kind="uniform")
    say(f"[staged windows] {kind} detector {ndet} of {ddet} mm")
    got = Plan(w.geometry_dict(), w.angles).backproject(torch.from_numpy(y).to(DEV), kind)
    ref = orc.bp(orc.Geometry.from_dict(w.geometry_dict()), w.angles, y.astype(np.float64),
                 orc.W_FDK if kind == "fdk" else orc.W_PM)
    assert rel_l2(got.cpu().numpy(), ref) <= TOL_BP
    # 16-bit projections take the converting copy: the same taps, bit for bit, of the same values
    h = torch.from_numpy(y).to(DEV).half()
    plan = Plan(w.geometry_dict(), w.angles)
    assert torch.equal(plan.backproject(h, kind, out_dtype=torch.float32),
                       plan.backproject(h.float(), kind, out_dtype=torch.float32))
