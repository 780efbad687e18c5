"""Tables that are symmetric but for one point (and its images under the other symmetry):
the plan may take no symmetry that the table does not have.  Without the mirror
symmetry the schedule names the general path; without the exchange of kx and ky the map
is that of the window on all points, bit for bit."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH

pytestmark = pytest.mark.gpu


def symmetric_table(n, seed=5):
    rng = np.random.Generator(np.random.PCG64(seed))
    q = rng.uniform(-0.7, 0.8, size=(n // 2 + 1, n // 2 + 1))
    q = q + q.T
    i = np.minimum(np.arange(n), n - np.arange(n))
    return q[i][:, i]


def plan_map(table, name="eps_table"):
    n = table.shape[0]
    kw = dict(eps_table=symmetric_table(n), mu=0.1, nkx=n, nky=n, neps=16, emin=-1.6, emax=1.6, gamma=0.2,
              omega=np.array([1, 5]) * 0.2, precision=LH.LINDHARD_FP64)
    kw[name] = table
    plan = LH.Plan(**kw)
    out = plan.exec().cpu()
    s = plan.info.schedule.decode()
    plan.close()
    return out, " even " in s


@pytest.mark.parametrize("name", ["eps_table", "rho_table"])
@pytest.mark.parametrize("n", [128, 131, 200])
def test_mirror(n, name):
    h = n // 2
    for y, x in ((0, 1), (1, 0), (3, h + 1), (h, 1), (h + 1, h), (n - 1, n - 1), (h, n - 1), (n - 1, 0), (0, n - 1)):
        t = symmetric_table(n) + 2.0
        assert plan_map(t, name)[1]
        t[y, x] += 1e-12
        assert not plan_map(t, name)[1]


@pytest.mark.parametrize("name", ["eps_table", "rho_table"])
@pytest.mark.parametrize("n", [128, 131, 200])
def test_exchange(n, name, monkeypatch):
    h = n // 2
    for y, x in ((0, 1), (1, 0), (31, 32), (32, 31), (33, 2), (h, 0), (0, h), (h, h - 1), (h - 1, h), (h, 32)):
        t = symmetric_table(n) + 2.0
        for yy in {y, (n - y) % n}:
            for xx in {x, (n - x) % n}:
                t[yy, xx] += 0.3
        monkeypatch.delenv("LINDHARD_SYMMETRY", raising=False)
        got, even = plan_map(t, name)
        monkeypatch.setenv("LINDHARD_SYMMETRY", "mirror")
        assert even and torch.equal(got, plan_map(t, name)[0])
