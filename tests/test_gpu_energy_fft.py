"""The general path's energy window by FFT against the direct form, for every
transform length (4 to 2048 energies) and at the edges of its rules: windows
whose occupied or unoccupied part is more than half of the transform, lags up to
and past half of it (RPA plans keep all), single lags, grids of any size.
Tolerance: the sum of both forms' tolerances of the hot path."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH

pytestmark = pytest.mark.gpu

TOL = {LH.LINDHARD_FP64: 1e-11, LH.LINDHARD_FP32C: 1e-5}
PRECS = [LH.LINDHARD_FP64, LH.LINDHARD_FP32C]


def both_forms(cfg, monkeypatch, rpa=False):
    maps = {}
    for form in ("direct", "fft"):
        monkeypatch.setenv("LINDHARD_WINDOW", form)
        plan = LH.Plan(**cfg)
        assert " P3 %s " % form in plan.info.schedule.decode()
        out = [plan.exec()]
        if rpa:
            out += list(plan.rpa(0.5))
        maps[form] = [o.double().cpu() for o in out]
        plan.close()
    return max(float((a - b).abs().max() / b.abs().max()) for a, b in zip(maps["fft"], maps["direct"]))


def config(prec, neps, lags, shape=(16, 8), emin=-1.6, emax=1.6, **kw):
    rng = np.random.Generator(np.random.PCG64(neps))
    tab = rng.uniform(-1.2, 1.4, size=(shape[1], shape[0]))
    return dict(eps_table=tab, mu=0.0, nkx=shape[0], nky=shape[1], neps=neps, emin=emin, emax=emax, gamma=0.1,
                omega=np.asarray(list(lags), dtype=np.float64) * ((emax - emin) / neps), precision=prec, **kw)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("neps", [4, 8, 16, 32, 64, 128, 256, 512, 1024, 2048])
def test_lengths(prec, neps, monkeypatch):
    half = neps // 2
    assert both_forms(config(prec, neps, {1, 2, half - 1, half}), monkeypatch) <= 2 * TOL[prec]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("neps", [64, 128, 512])
@pytest.mark.parametrize("window", [(-0.3, 2.9), (-2.9, 0.3), (-1.6, 1.6)])
def test_uneven_windows_and_long_lags(prec, neps, window, monkeypatch):
    lags = {1, neps // 2 + 1, 3 * neps // 4, neps - 1, neps}
    cfg = config(prec, neps, lags, emin=window[0], emax=window[1])
    assert both_forms(cfg, monkeypatch) <= 2 * TOL[prec]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape", [(16, 8), (13, 11)])
def test_rpa_and_any_size(prec, shape, monkeypatch):
    cfg = config(prec, 64, [3, 20, 45], shape=shape, want_rpa=True)
    assert both_forms(cfg, monkeypatch, rpa=True) <= 2 * TOL[prec]


@pytest.mark.parametrize("prec", PRECS)
def test_single_lag(prec, monkeypatch):
    assert both_forms(config(prec, 64, [1]), monkeypatch) <= 2 * TOL[prec]
