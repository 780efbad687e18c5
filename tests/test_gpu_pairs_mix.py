"""Band pairs on the rank-1 matrix window (it reads the bands' spectra in place and
mixes the unoccupied ones while staging) against the direct window, which works
on spliced copies: constant weights with zeros among them, |M(Q)|^2 maps, one to
four bands, lag ranges at the edges of the 16-lag tiles, uneven windows.
Tolerance: the sum of both forms' tolerances of the hot path."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH
from paper_1208_3210_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-5
WEIGHTS = {
    "full": lambda nb: np.arange(1.0, nb * nb + 1).reshape(nb, nb) / 4,
    "diagonal": lambda nb: np.eye(nb),
    "one_row": lambda nb: np.vstack([np.zeros((nb - 1, nb)), np.full((1, nb), 0.5)]),
    "one_column": lambda nb: np.hstack([np.full((nb, 1), 2.0), np.zeros((nb, nb - 1))]),
}


def both(cfg, monkeypatch):
    maps = {}
    for form in ("direct", "mfma4"):
        monkeypatch.setenv("LINDHARD_EVEN_WINDOW", form)
        plan = LH.Plan(precision=LH.LINDHARD_FP32C, **cfg)
        assert " P3 %s " % form in plan.info.schedule.decode()
        first = plan.exec().clone()
        assert torch.equal(first, plan.exec())  # nothing of a call is left for the next
        maps[form] = first.double().cpu()
        plan.close()
    a, b = maps["mfma4"], maps["direct"]
    return float((a - b).abs().max() / b.abs().max())


def config(n, nb, lags, emin=-1.6, emax=1.6, neps=64, **kw):
    return dict(eps_table=W.multiband_tables(n, nb), n_bands=nb, mu=0.05, nkx=n, nky=n, neps=neps, emin=emin, emax=emax,
                gamma=0.08, omega=np.asarray(list(lags), dtype=np.float64) * ((emax - emin) / neps), **kw)


@pytest.mark.parametrize("weights", sorted(WEIGHTS))
@pytest.mark.parametrize("nb", [1, 2, 4])
@pytest.mark.parametrize("lags", [[1], range(1, 17), range(3, 34), [60, 63]])
def test_constant_weights(nb, weights, lags, monkeypatch):
    assert both(config(32, nb, lags, pair_weight=WEIGHTS[weights](nb)), monkeypatch) <= 2 * TOL


@pytest.mark.parametrize("window", [(-0.4, 2.8), (-2.8, 0.4)])
def test_uneven_windows(window, monkeypatch):
    cfg = config(64, 2, range(1, 40), emin=window[0], emax=window[1], pair_weight=WEIGHTS["full"](2))
    assert both(cfg, monkeypatch) <= 2 * TOL


@pytest.mark.parametrize("nb", [2, 3])
def test_maps(nb, monkeypatch):
    n = 32
    rng = np.random.Generator(np.random.PCG64(7))
    m2 = rng.uniform(0.0, 1.0, size=(nb, nb, n, n))
    m2[0, nb - 1] = 0.0
    assert both(config(n, nb, range(1, 20), pair_m2=m2), monkeypatch) <= 2 * TOL


def test_exchange_symmetric_bands(monkeypatch):
    n = 128
    tabs = W.multiband_tables(n, 2)
    cfg = config(n, 2, range(1, 20), pair_weight=WEIGHTS["full"](2))
    cfg["eps_table"] = 0.5 * (tabs + tabs.transpose(0, 2, 1))
    assert both(cfg, monkeypatch) <= 2 * TOL
