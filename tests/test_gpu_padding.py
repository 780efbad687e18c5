"""Band pairs symmetric under the exchange of kx and ky, called many times on one plan:
the half window leaves the padding columns of the last tile alone, and the inverse
column pass runs in place beside them, so nothing of a call may stay there for the
next one (or of one pair's map for the next pair's).  Every call must equal the
first bit for bit; the first against the direct window, which works on copies, with the
sum of both forms' tolerances of the hot path."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH
from paper_1208_3210_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {LH.LINDHARD_FP64: 1e-11, LH.LINDHARD_FP32C: 1e-5}
CALLS = 40


def symmetric(n, nb):
    t = W.multiband_tables(n, nb)
    return 0.5 * (t + t.transpose(0, 2, 1))


def config(n, nb, nlag=19, neps=64, w=1.6, **kw):
    return dict(eps_table=symmetric(n, nb), n_bands=nb, mu=0.05, nkx=n, nky=n, neps=neps, emin=-w, emax=w, gamma=0.08,
                omega=np.arange(1, nlag + 1) * (2 * w / neps), **kw)


def check(cfg, prec, form, monkeypatch):
    maps = {}
    for f, calls in ((form, CALLS), ("direct", 1)):
        monkeypatch.setenv("LINDHARD_EVEN_WINDOW", f)
        plan = LH.Plan(precision=prec, **cfg)
        assert " P3 %s " % f in plan.info.schedule.decode()
        first = plan.exec().clone()
        again = torch.empty_like(first)
        for _ in range(calls - 1):
            again.fill_(float("nan"))
            plan.exec(again)
            assert torch.equal(first, again)
        maps[f] = first.double().cpu()
        plan.close()
    assert float((maps[form] - maps["direct"]).abs().max() / maps["direct"].abs().max()) <= 2 * TOL[prec]


FORMS = [(LH.LINDHARD_FP32C, "mfma4"), (LH.LINDHARD_FP32C, "mfma"), (LH.LINDHARD_FP64, "mfma")]


@pytest.mark.parametrize("prec,form", FORMS)
@pytest.mark.parametrize("n,nb", [(128, 2), (256, 2), (512, 3), (1024, 2)])
def test_pair_weights(n, nb, prec, form, monkeypatch):
    w = np.arange(1.0, nb * nb + 1).reshape(nb, nb) / 4
    check(config(n, nb, pair_weight=w), prec, form, monkeypatch)


@pytest.mark.parametrize("prec,form", FORMS)
@pytest.mark.parametrize("n,nb", [(128, 3), (256, 4), (1024, 2)])
def test_pair_maps(n, nb, prec, form, monkeypatch):
    m2 = np.random.Generator(np.random.PCG64(11)).uniform(0.0, 1.0, size=(nb, nb, n, n))
    check(config(n, nb, pair_m2=m2), prec, form, monkeypatch)
