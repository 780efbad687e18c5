"""Grids of any size with zones: the images of a row are dealt out to several blocks when
rows and omegas are few.  The same omegas among so many that one block writes all of a
row's images, with omegas outside the window (planes of zeros) in both: equal bit for
bit, and the images of a map without the orbital are the first zone's."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [LH.LINDHARD_FP64, LH.LINDHARD_FP32C])
@pytest.mark.parametrize("ff", [0, 1])
@pytest.mark.parametrize("zones", [(1, 1), (3, 1), (1, 3), (3, 5), (7, 7)])
@pytest.mark.parametrize("nkx,nky", [(5, 33), (33, 6), (47, 47)])
def test_images(nkx, nky, zones, ff, prec):
    d = 3.2 / 64
    few = np.array([1, 2.5, 9, 63, 80.0])
    many = np.concatenate([few, np.linspace(1, 70, 2100)])
    kw = dict(t=0.4, tp=-0.1, tpp=0.04, mu=0.1, nkx=nkx, nky=nky, neps=64, emin=-1.6, emax=1.6, gamma=0.09,
              omega_interp=True, zones=zones, ff_kind=ff, ff_width=0.6 if ff else 0.0, precision=prec)
    maps = []
    for om in (few, many):
        plan = LH.Plan(omega=om * d, **kw)
        out = plan.empty().fill_(float("nan"))
        maps.append(plan.exec(out)[:len(few)].clone())
        assert not torch.isnan(out).any()
        plan.close()
    assert torch.equal(maps[0], maps[1])
    if not ff:
        m = maps[0].reshape(len(few), zones[1], nky, zones[0], nkx)
        cy, cx = zones[1] // 2, zones[0] // 2
        assert torch.equal(m, m[:, cy:cy + 1, :, cx:cx + 1].expand_as(m))
