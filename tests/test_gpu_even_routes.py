"""The even path's builder and column passes at the lines between the full and the
half-work transform (numbers of rows, tiles and slices), against the general complex
transforms of the same library: both sides of each line, and a batch whose plans of one
grid lie on both sides (each equals its plan run alone, bit for bit).
Tolerance: the sum of both sides' tolerances of the hot path."""
import numpy as np
import pytest
import torch

from paper_1208_3210_amd import lindhard as LH
from paper_1208_3210_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {LH.LINDHARD_FP64: 1e-11, LH.LINDHARD_FP32C: 1e-5}
PRECS = [LH.LINDHARD_FP64, LH.LINDHARD_FP32C]


def config(shape, lags, prec, neps=128, **kw):
    return dict(**W.BAND1, filling=1.15, nkx=shape[0], nky=shape[1], neps=neps, emin=-2.0, emax=2.0, gamma=0.05,
                omega=W.lag_omegas(neps, -2.0, 2.0, lags), precision=prec, **kw)


# rows: 1024 x 256 has 17 blocks of 8 rows (30 pairs of slices are too few, 31 enough),
# 2048 x 128 too few rows in FP32 and 17 blocks of 4 in FP64; columns: 64 x 2048 has 9
# tiles in FP64 (25 slices are too few, 26 enough)
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape,lags", [((1024, 256), [30]), ((1024, 256), [31]), ((2048, 128), [30]), ((2048, 128), [62]),
                                        ((64, 2048), [12]), ((64, 2048), [13]), ((64, 2048), range(1, 25)),
                                        ((64, 2048), range(1, 28)), ((4096, 16), [1, 5]), ((8, 4096), [1, 5])])
def test_lines(shape, lags, prec, monkeypatch):
    maps = {}
    for path in ("off", "on"):
        monkeypatch.setenv("LINDHARD_SYMMETRY", path)
        plan = LH.Plan(**config(shape, lags, prec))
        assert (" even " in plan.info.schedule.decode()) == (path == "on")
        maps[path] = plan.exec().double().cpu()
        plan.close()
    assert float((maps["on"] - maps["off"]).abs().max() / maps["off"].abs().max()) <= 2 * TOL[prec]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape", [(1024, 256), (64, 2048)])
def test_batch_across_the_lines(shape, prec):
    cfgs = [config(shape, range(1, k), prec) for k in (3, 12, 30, 33, 40, 60)]
    plans = [LH.Plan(**c) for c in cfgs]
    alone = [p.exec().clone() for p in plans]
    for _ in range(3):
        outs = LH.exec_batch(plans)
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(alone, outs))
    for p in plans:
        p.close()
