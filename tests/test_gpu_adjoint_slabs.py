"""The exact adjoint of a volume cut into slabs is bit for bit the whole one's: slabs that start on odd and on
even slices, of fewer and of more than 64 slices, with one and with two slab buffers, where 2, 3 and 4 detector
rows can meet two neighbouring voxels (they are taken in pairs), where more can, and in volumes of up to 64
slices with few columns (taken one by one) and with many (in pairs)."""
import pytest
import torch

from _helpers import say
from paper_1905_03748_amd import inputs
from paper_1905_03748_amd._abi import CtError
from paper_1905_03748_amd.operators import Plan

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _cap(plan, n_slabs):
    """The least cap (in steps of a slice) with which the planner makes n_slabs slabs."""
    nz, ny, nx = plan.vol_shape
    for h in range(4 * nz):
        cap = (64 << 20) + h * nx * ny * 4
        try:
            if plan.ooc_plan(2, cap_bytes=cap)["n_slabs"] == n_slabs:
                return cap
        except CtError:   # below the least
            continue
    raise AssertionError(f"no cap gives {n_slabs} slabs")


# columns, slices, slice height, rows, row pitch
@pytest.mark.parametrize("nxy,nz,dz,nv,dv", [((25, 24), 259, 0.8, 200, 2.6), ((25, 24), 259, 0.8, 300, 1.4),
                                             ((25, 24), 259, 0.8, 420, 0.8), ((25, 24), 259, 0.8, 500, 0.6),
                                             ((25, 24), 61, 1.0, 71, 1.6), ((81, 80), 61, 1.0, 71, 1.6)])
@pytest.mark.parametrize("n_slabs", [3, 4, 9])
def test_adjoint_slabs_bitwise(nxy, nz, dz, nv, dv, n_slabs, monkeypatch):
    w = inputs.Workload("adj_slabs", nxy + (nz,), (1.4, 1.5, dz), (27, nv), (1.3, dv), 11, 10, 3,
                        off_origin=(2.0, -1.0, 0.3), off_detector=(0.31, 0.0))
    plan = Plan(w.geometry_dict(), w.angles + 0.1)
    y = inputs.random_array((11, nv, 27), 6, kind="uniform")
    ref = plan.backproject(torch.from_numpy(y).to(DEV), "adjoint").cpu()
    for buffers in ("1", "2"):
        monkeypatch.setenv("CT_OOC_SLAB_BUFFERS", buffers)
        cap = _cap(plan, n_slabs)
        out = torch.full(plan.vol_shape, -7.0)
        say(f"[adjoint slabs] {nz} slices, {n_slabs} slabs, {buffers} buffers")
        st = plan.backproject_host(torch.from_numpy(y), out, "adjoint", cap_bytes=cap)
        assert st["n_slabs"] == n_slabs, st
        assert torch.equal(out, ref), (st, float((out - ref).abs().max()))
