"""The column-major OS-SART update against the CPU FP64 oracle where a wave's heights take 1, 2, 4 or more
groups of 64 (the last ones partly or wholly past the column), where they leave the detector above and below,
where many detector rows lie between two heights, and where so many do that the general update takes over."""
import numpy as np
import pytest
import torch

from _helpers import TOL_BP, rel_l2, say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("nz,dz,ndet,ddet", [
    (1, 1.0, (21, 9), (2.4, 2.0)), (63, 0.9, (21, 70), (2.4, 1.7)), (64, 0.9, (22, 40), (2.4, 1.6)),
    (65, 0.9, (21, 101), (2.4, 1.3)), (130, 0.5, (21, 90), (2.4, 1.2)), (200, 0.4, (20, 120), (2.4, 1.1)),
    (300, 0.3, (21, 97), (2.4, 1.5)), (330, 0.3, (10, 97), (2.4, 1.5)), (90, 1.0, (21, 300), (2.4, 0.6)),
    (40, 4.0, (19, 600), (2.4, 0.11)), (40, 4.0, (5, 3000), (9.0, 0.1))])
def test_os_sart_update_rows(orc, nz, dz, ndet, ddet):
    w = inputs.Workload("sart_rows", (14, 13, nz), (1.5, 1.6, dz), ndet, ddet, 23, 10, 5, off_origin=(1.1, -0.6, 3.0),
                        off_detector=(0.4, -0.3))
    say(f"[sart rows] {nz} slices of {dz}, detector {ndet} of {ddet}")
    og = orc.Geometry.from_dict(w.geometry_dict())
    vol = np.random.default_rng(3).uniform(0, 1, w.nvox[::-1])
    b = orc.siddon_fwd(og, w.angles, vol).astype(np.float32)
    got = Plan(w.geometry_dict(), w.angles).sart(torch.from_numpy(b).to(DEV), 2, lam=0.8, block=18)
    ref = orc.os_sart(og, w.angles, b.astype(np.float64), 2, block=18, lam=0.8)
    assert rel_l2(got.cpu().numpy(), ref) <= TOL_BP
