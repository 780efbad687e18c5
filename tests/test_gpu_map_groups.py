"""The RPA path's maps take columns of zones in groups that depend on the number of
omegas: the maps of a few omegas among many equal those of the few alone, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [LH.LINDHARD_FP64, LH.LINDHARD_FP32C])
@pytest.mark.parametrize("zones", [(1, 1), (3, 1), (5, 3), (7, 1), (9, 1), (11, 3)])
@pytest.mark.parametrize("nkx,nky", [(16, 8), (6, 9), (64, 32)])
def test_groups(nkx, nky, zones, prec):
    d = 3.2 / 32
    few = np.array([1, 2.5, 9])
    many = np.concatenate([few, np.arange(1, 30)])
    kw = dict(t=0.4, tp=-0.1, tpp=0.04, mu=0.1, nkx=nkx, nky=nky, neps=32, emin=-1.6, emax=1.6, gamma=0.09,
              omega_interp=True, zones=zones, ff_kind=1, ff_width=0.6, precision=prec, want_rpa=True)
    maps = []
    for om in (few, many):
        plan = LH.Plan(omega=om * d, **kw)
        maps.append([plan.exec()] + list(plan.rpa(0.8)) + list(plan.rpa_coulomb(0.5)))
        torch.cuda.synchronize()
        assert not any(torch.isnan(m).any() for m in maps[-1])
        plan.close()
    for a, b in zip(*maps):
        assert torch.equal(a, b[:len(few)])


def test_rows_beyond_one_launch():
    """More than 2^19 blocks of rows (three dimensions, 16383 zones along y): every zone
    image equals the map of one zone."""
    nkx, nky, nkz, zy = 8, 4, 256, 16383
    eps = np.random.Generator(np.random.PCG64(4)).uniform(-0.8, 0.8, size=(nkz, nky, nkx))
    kw = dict(eps_table=eps, nkz=nkz, mu=0.1, nkx=nkx, nky=nky, neps=8, emin=-1.6, emax=1.6, gamma=0.2,
              omega=[0.8], want_rpa=True, precision=LH.LINDHARD_FP32C)
    one, many = LH.Plan(**kw), LH.Plan(zones=(1, zy), **kw)
    for a, b in zip([one.exec()] + list(one.rpa(0.8)), [many.exec()] + list(many.rpa(0.8))):
        a = a.reshape(nkz, 1, nky, nkx)
        assert torch.equal(b.reshape(nkz, zy, nky, nkx), a.expand(nkz, zy, nky, nkx))
    one.close()
    many.close()
