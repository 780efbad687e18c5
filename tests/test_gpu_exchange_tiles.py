"""The matrix window with few points per block (four: half a tile row in FP32) on bands
symmetric under the exchange of kx and ky, against the window on all points of the same
library, on square grids of powers of two and of any size.  Four points per block are
what is taken without timing, and the only fit at many energies and long lags.
Tolerance: the sum of both sides' tolerances of the hot path."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH

pytestmark = pytest.mark.gpu

TOL = {LH.LINDHARD_FP64: 1e-11, LH.LINDHARD_FP32C: 1e-5}
PRECS = [LH.LINDHARD_FP32C, LH.LINDHARD_FP64]


def symmetric_table(n, seed=5):
    rng = np.random.Generator(np.random.PCG64(seed))
    q = rng.uniform(-0.7, 0.8, size=(n // 2 + 1, n // 2 + 1))
    q = q + q.T
    i = np.minimum(np.arange(n), n - np.arange(n))
    return q[i][:, i]


def both(cfg, prec, schedule, monkeypatch):
    monkeypatch.setenv("LINDHARD_EVEN_WINDOW", "mfma")
    maps = {}
    for path in ("exchange", "mirror"):
        monkeypatch.setenv("LINDHARD_SYMMETRY", path)
        plan = LH.Plan(precision=prec, **cfg)
        assert schedule in plan.info.schedule.decode()
        out = [plan.exec()]
        if cfg.get("want_rpa"):
            out += list(plan.rpa(0.8))
        maps[path] = [o.double().cpu() for o in out]
        plan.close()
    for a, b in zip(maps["exchange"], maps["mirror"]):
        assert float((a - b).abs().max() / b.abs().max()) <= 2 * TOL[prec]


def config(n, lags, neps, w=1.6, **kw):
    return dict(eps_table=symmetric_table(n), mu=0.1, nkx=n, nky=n, neps=neps, emin=-w, emax=w, gamma=0.09,
                omega=np.asarray(lags, dtype=np.float64) * (2 * w / neps), **kw)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("rpa", [False, True])
@pytest.mark.parametrize("n", [16, 33, 128, 129, 150])
def test_four_points(n, rpa, prec, monkeypatch):
    monkeypatch.setenv("LINDHARD_AUTOTUNE", "0")
    cfg = config(n, range(1, 20), 64)
    if rpa:
        cfg.update(want_rpa=True, zones=(3, 1))
    both(cfg, prec, " P3 mfma TR4 ", monkeypatch)


MANY = [(1024, [3, 300, 511], False), (1024, [1, 40], True), (2048, [5, 800, 1023], False)]


# (2048 energies and 1019 lags in FP64 do not fit any width of the matrix window)
@pytest.mark.parametrize("prec,neps,lags,rpa", [(p, *m) for p in PRECS for m in MANY
                                                if p == LH.LINDHARD_FP32C or m[0] < 2048])
@pytest.mark.parametrize("n", [32, 47, 128])
def test_many_energies(n, neps, lags, rpa, prec, monkeypatch):
    """The widths that the timing chooses from (eight and four points, or four alone)."""
    cfg = config(n, lags, neps)
    if rpa:
        cfg.update(want_rpa=True)
    both(cfg, prec, " P3 mfma TR", monkeypatch)
