"""Bands symmetric under the exchange of kx and ky: the window on half of the
real-space points against the FP64 oracle and against the same library with the
exchange symmetry not used, for every window form, at the sizes where a tile, a
unit of four rows or a block of points ends, on square grids of any size.
Tolerances as for the hot path; against the other path the sum of both sides'."""
import numpy as np
import pytest
import torch

import oracle
from paper_1208_3210_amd import lindhard as LH
from paper_1208_3210_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {LH.LINDHARD_FP64: 1e-11, LH.LINDHARD_FP32C: 1e-5}
PRECS = [LH.LINDHARD_FP64, LH.LINDHARD_FP32C]
WINDOWS = {LH.LINDHARD_FP64: ["direct", "mfma"], LH.LINDHARD_FP32C: ["direct", "mfma", "mfma4"]}
PW = [(p, w) for p in PRECS for w in WINDOWS[p]]


def normwise(got, ref):
    return float((got.double() - ref.double()).abs().max() / ref.double().abs().max())


def symmetric_table(n, seed=5):
    """Random, mirror symmetric in both axes and under their exchange."""
    rng = np.random.Generator(np.random.PCG64(seed))
    q = rng.uniform(-0.7, 0.8, size=(n // 2 + 1, n // 2 + 1))
    q = q + q.T
    i = np.minimum(np.arange(n), n - np.arange(n))
    return q[i][:, i]


def config(n, lags, neps=32, w=1.6, **kw):
    return dict(dict(eps_table=symmetric_table(n), mu=0.1, nkx=n, nky=n, neps=neps, emin=-w, emax=w, gamma=0.09,
                     omega=np.asarray(lags, dtype=np.float64) * (2 * w / neps)), **kw)


@pytest.mark.parametrize("prec,window", PW)
@pytest.mark.parametrize("n", [16, 17, 32, 47])
def test_against_oracle(prec, window, n, monkeypatch):
    monkeypatch.setenv("LINDHARD_EVEN_WINDOW", window)
    monkeypatch.setenv("LINDHARD_SYMMETRY", "exchange")
    cfg = config(n, range(1, 20))
    full = oracle.chi_full(cfg["eps_table"] - 0.1, 32, -1.6, 1.6, 0.09, np.arange(1, 20))
    ref = torch.from_numpy(oracle.extend(full, 1, 1, 0, 0.0))
    plan = LH.Plan(precision=prec, **cfg)
    assert normwise(plan.exec().cpu(), ref) <= TOL[prec]
    plan.close()


FORMS = {
    "one_lag": dict(lags=[5]),
    "sparse_lags": dict(lags=[0, 3, 17, 40]),
    "asymmetric_window": dict(lags=range(1, 30), emin=-0.6, emax=2.6),
    "rpa": dict(lags=[1, 4, 9], want_rpa=True, zones=(3, 1)),
    "interp": dict(lags=[0.5, 6.25], omega_interp=True),
    "rho": dict(lags=range(1, 12), rho=True, k_zones=2),
    "bands": dict(lags=range(1, 12), nb=2),
    "pairs": dict(lags=range(1, 12), nb=2, pair_weight=np.array([[1.0, 0.3], [0.0, 2.0]])),
}


@pytest.mark.parametrize("prec,window", PW)
@pytest.mark.parametrize("form", sorted(FORMS))
@pytest.mark.parametrize("n", [32, 64, 90])
def test_forms_against_mirror_path(prec, window, form, n, monkeypatch):
    f = dict(FORMS[form])
    if "nb" in f and n & (n - 1):
        n = 16  # several bands: powers of two
    cfg = config(n, f.pop("lags"))
    if f.pop("rho", False):
        f["rho_table"] = W.density_s(n, n, f["k_zones"], 0.4)
    nb = f.pop("nb", 1)
    if nb > 1:
        cfg["eps_table"] = np.stack([symmetric_table(n, 5), symmetric_table(n, 6)])
        f["n_bands"] = nb
    cfg.update(f)
    monkeypatch.setenv("LINDHARD_EVEN_WINDOW", window)
    maps = {}
    for path in ("mirror", "exchange"):
        monkeypatch.setenv("LINDHARD_SYMMETRY", path)
        plan = LH.Plan(precision=prec, **cfg)
        out = [plan.exec()]
        if cfg.get("want_rpa"):
            out += list(plan.rpa(0.8))
        maps[path] = [o.cpu() for o in out]
        plan.close()
    for a, b in zip(maps["exchange"], maps["mirror"]):
        assert normwise(a, b) <= 2 * TOL[prec]


@pytest.mark.parametrize("prec", PRECS)
def test_batch_mixes_symmetric_and_other_bands(prec, monkeypatch):
    """Both kinds of one grid in one batch: each equals its plan run alone, bit for bit."""
    monkeypatch.setenv("LINDHARD_SYMMETRY", "exchange")
    cfgs = [config(64, range(1, 16)) for _ in range(2)]
    for s in (1, 2):
        t = symmetric_table(64, 8 + s)
        t[:, :] += 0.1 * np.cos(2 * np.pi * np.minimum(np.arange(64), 64 - np.arange(64)) / 64)[None, :]
        cfgs.append(dict(config(64, range(1, 16)), eps_table=t))
    plans = [LH.Plan(precision=prec, **c) for c in cfgs]
    alone = [p.exec().clone() for p in plans]
    for _ in range(2):
        outs = LH.exec_batch(plans)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(alone, outs))
    for p in plans:
        p.close()
