"""The staged exact adjoint of tilted views at each row pitch of its LDS windows: the narrow one (up to 41 columns),
the middle one (42 to 49) with windows of few rows, which the wide pitch would hold too, and of more rows, which only
the middle one holds, and the wide one; against the kernel without staging and the CPU FP64 oracle."""
import numpy as np
import pytest
import torch

from _helpers import TOL_BP, rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# pixel size (mm) for the host's window bound (columns x rows) of the 1.1 mm grid
@pytest.mark.parametrize("ddet,window", [((1.8, 1.3), "31 x 27"), ((1.2, 1.6), "44 x 23"), ((1.15, 1.3), "46 x 27"),
                                         ((1.2, 1.1), "44 x 32"), ((1.15, 1.0), "46 x 34"), ((1.25, 0.85), "43 x 40"),
                                         ((1.0, 1.6), "52 x 23")])
def test_staged_adjoint_pitches(orc, ddet, window, monkeypatch):
    ndet = (int(70 / ddet[0]), int(66 / ddet[1]))
    w = inputs.Workload("pitch", (37, 34, 35), (1.1, 1.1, 1.1), ndet, ddet, 13, 10, 5, off_origin=(1.1, -0.6, 0.8),
                        off_detector=(0.4, -0.3))
    views = inputs.carm_views(w.DSO, w.DSD, w.angles + 0.2, 17, tilt_deg=10.0, jitter_mm=5.0, orbit_tilt_deg=5.0)
    plan = Plan(w.geometry_dict(), views)
    y = inputs.random_array((13, ndet[1], ndet[0]), 8, kind="uniform")
    yd = torch.from_numpy(y).to(DEV)
    say(f"[pitch] window {window}, detector {ndet} of {ddet}")
    a = plan.backproject(yd, "adjoint")
    monkeypatch.setenv("CT_VIEWS_ADJ_DIRECT", "1")
    b = plan.backproject(yd, "adjoint")
    monkeypatch.delenv("CT_VIEWS_ADJ_DIRECT")
    assert not torch.equal(a, b), "the staged kernel did not run"
    assert rel_l2(a.cpu().numpy(), b.cpu().numpy()) <= 2e-6
    ref = orc.siddon_adj(orc.Geometry.from_dict(w.geometry_dict()), views, y.astype(np.float64))
    assert rel_l2(a.cpu().numpy(), ref) <= TOL_BP
    h = torch.from_numpy(y).to(DEV).half()
    assert rel_l2(plan.backproject(h, "adjoint", out_dtype=torch.float32).cpu().numpy(),
                  plan.backproject(h.float(), "adjoint").cpu().numpy()) <= 1e-6
