"""The even path's builder and column passes on the half-work transform (axes of
1024 points and more; FP64 columns from 512) against the general complex
transforms of the same library: each axis length alone and both at once, odd
numbers of energy slices, momentum densities, several bands (accumulated
builder passes) and empty planes; a sampled comparison with the FP64 oracle.
Tolerance: the sum of both sides' tolerances of the hot path."""
import numpy as np
import pytest
import torch

import oracle
from paper_1208_3210_amd import lindhard as LH
from paper_1208_3210_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {LH.LINDHARD_FP64: 1e-11, LH.LINDHARD_FP32C: 1e-5}
PRECS = [LH.LINDHARD_FP64, LH.LINDHARD_FP32C]


def normwise(got, ref):
    return float((got.double() - ref.double()).abs().max() / ref.double().abs().max())


def both_paths(cfg, monkeypatch):
    maps = {}
    for path in ("off", "on"):
        monkeypatch.setenv("LINDHARD_SYMMETRY", path)
        plan = LH.Plan(**cfg)
        assert (" even " in plan.info.schedule.decode()) == (path == "on")
        maps[path] = plan.exec().cpu()
        plan.close()
    return maps["on"], maps["off"]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape", [(1024, 4), (4, 1024), (2048, 16), (16, 2048), (4096, 8), (8, 4096), (64, 512),
                                   (1024, 512), (1024, 1024)])
def test_axis_lengths(prec, shape, monkeypatch):
    nkx, nky = shape
    cfg = dict(**W.BAND1, filling=1.15, nkx=nkx, nky=nky, neps=32, emin=-2.0, emax=2.0, gamma=0.05,
               omega=W.lag_omegas(32, -2.0, 2.0, range(1, 12)), precision=prec)
    a, b = both_paths(cfg, monkeypatch)
    assert normwise(a, b) <= 2 * TOL[prec]


FORMS = {
    "odd_slices": dict(lags=range(1, 20), emin=-0.7, emax=2.5),
    "one_lag": dict(lags=[1]),
    "empty_plane": dict(lags=[0, 7, 64]),
    "rho": dict(lags=range(1, 9), rho=1, k_zones=4),
    "bands": dict(lags=range(1, 9), nb=3),
    "bands_rho": dict(lags=range(1, 9), nb=2, rho=2),
}


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("form", sorted(FORMS))
def test_forms(prec, form, monkeypatch):
    f = dict(FORMS[form])
    n, nky, neps = 1024, 1024, 32
    emin, emax = f.pop("emin", -1.6), f.pop("emax", 1.6)
    cfg = dict(**W.BAND1, filling=1.15, nkx=n, nky=nky, neps=neps, emin=emin, emax=emax, gamma=0.06, precision=prec,
               omega=np.asarray(f.pop("lags"), dtype=np.float64) * ((emax - emin) / neps))
    nb, rho = f.pop("nb", 1), f.pop("rho", 0)
    if nb > 1:
        cfg.update(eps_table=W.multiband_tables(n, nb), n_bands=nb)
    if rho:
        d = W.density_s(n, nky, f.get("k_zones", 1), 0.3)
        cfg["rho_table"] = np.stack([d * (1 + 0.5 * i) for i in range(nb)])
    cfg.update(f)
    a, b = both_paths(cfg, monkeypatch)
    assert normwise(a, b) <= 2 * TOL[prec]


@pytest.mark.parametrize("prec", PRECS)
def test_sampled_against_oracle(prec):
    n, neps = 1024, 32
    cfg = dict(**W.BAND1, mu=0.2, nkx=n, nky=8, neps=neps, emin=-2.0, emax=2.0, gamma=0.05,
               omega=W.lag_omegas(neps, -2.0, 2.0, range(1, 17)), precision=prec)
    xi = oracle.band_tb(W.BAND1["t"], W.BAND1["tp"], W.BAND1["tpp"], n, 8) - 0.2
    rng = np.random.Generator(np.random.PCG64(1))
    qx, qy, m = rng.integers(0, n, 40), rng.integers(0, 8, 40), rng.integers(1, 17, 40)
    ref = oracle.chi_pairs(xi, neps, -2.0, 2.0, 0.05, qx, qy, m)
    plan = LH.Plan(**cfg)
    out = plan.exec().double().cpu().numpy()
    got = out[m - 1, (qy + 4) % 8, (qx + n // 2) % n]
    assert np.abs(got - ref).max() <= TOL[prec] * np.abs(ref).max()
    plan.close()


def test_batch_equals_alone():
    cfgs = [dict(**W.BAND1, filling=1.0 + 0.05 * i, nkx=1024, nky=1024, neps=32, emin=-2.0, emax=2.0, gamma=0.05,
                 omega=W.lag_omegas(32, -2.0, 2.0, range(1, 5 + 4 * i)), precision=LH.LINDHARD_FP32C) for i in range(3)]
    plans = [LH.Plan(**c) for c in cfgs]
    alone = [p.exec().clone() for p in plans]
    for _ in range(3):
        outs = LH.exec_batch(plans)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(alone, outs))
    for p in plans:
        p.close()
