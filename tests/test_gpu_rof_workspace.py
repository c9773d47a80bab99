"""ROF on workspaces of a caller: four volumes are enough (two passes per iteration), six give one pass, the
size is never overrun, and the results agree bit for bit with those of the library's own scratch."""
import pytest
import torch

from _helpers import say
from paper_1905_03748_amd import _abi as A
from paper_1905_03748_amd.operators import _stream, rof, rof_workspace_bytes

DEV = "cuda:0"
SHAPE = (9, 21, 67)
VOLUME = -(-9 * 21 * 67 * 4 // 256) * 256


def _geo(shape):
    return dict(DSO=1000.0, DSD=1500.0, nVoxel=shape[::-1], dVoxel=(1.0, 1.0, 1.0), offOrigin=(0, 0, 0),
                nDetector=(8, 8), dDetector=(1.0, 1.0), offDetector=(0, 0), accuracy=0.5)


def test_rof_workspace_is_four_volumes():
    assert A.ct_rof_workspace_bytes(A.make_geometry(_geo(SHAPE))) == 4 * VOLUME
    assert rof_workspace_bytes(_geo(SHAPE)) == 6 * VOLUME
    big = _geo((1700, 1600, 1600))   # 17.4 GB a volume
    assert rof_workspace_bytes(big) == A.ct_rof_workspace_bytes(A.make_geometry(big)) == 4 * 1700 * 1600 * 1600 * 4


def test_rof_sized_refuses_a_short_workspace():
    g = A.make_geometry(_geo(SHAPE))
    with pytest.raises(A.CtError) as e:   # refused before any device work
        A.ct_rof_sized(g, 256, 1, 0.1, 0.08, 256, 4 * VOLUME - 1)
    assert e.value.status == A.CT_ERR_ARG


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ["rof", "ct_rof"])
@pytest.mark.parametrize("volumes", [4, 5, 6])
@pytest.mark.parametrize("niter", [0, 1, 6])
def test_rof_keeps_to_its_workspace(entry, volumes, niter):
    geo = _geo(SHAPE)
    f = torch.rand(SHAPE, generator=torch.Generator().manual_seed(7)).to(DEV)
    ref = rof(geo, f.clone(), niter, 0.1)
    say(f"[rof workspace] {entry}, {volumes} volumes, {niter} iterations")
    guard = 4096
    buf = torch.full((6 * VOLUME + guard,), 0xA5, dtype=torch.uint8, device=DEV)
    x = f.clone()
    if entry == "rof":
        rof(geo, x, niter, 0.1, workspace=buf[:volumes * VOLUME])
    else:
        A.ct_rof(A.make_geometry(geo), x.data_ptr(), niter, 0.1, 1.0 / 12.0, buf.data_ptr(), _stream())
    assert torch.equal(x, ref)
    held = volumes if entry == "rof" else 4   # ct_rof knows its buffer by the least size alone
    assert bool((buf[held * VOLUME:] == 0xA5).all())
