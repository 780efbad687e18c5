"""The extended maps of the RPA path (Im chi, Re chi, chi_RPA) where their kernel
changes form: rows that allow 16-byte accesses and rows that do not, one zone
and several, more zones than a thread holds at once, rows of several segments,
outputs at addresses that are not 16-byte aligned, omitted outputs, omegas between
lags.  The one-zone plan without form factor of the same problem gives the
first-zone values; tiling, the form factor and chi / (1 - V chi) are
done in FP64 on the host.  Tolerance per value: Im and Re are one product rounded to
the output type (plus the rounding of the first-zone values): 2 ulp; chi_RPA of the
returned Im and Re is one FP64 expression rounded once: 1 ulp and 16 FP64 ulps
of its largest term, times the amplification of the denominator's rounding."""
import numpy as np
import pytest
import torch

import oracle
from paper_1208_3210_amd import lindhard as LH
from paper_1208_3210_amd import workloads as W

pytestmark = pytest.mark.gpu

PRECS = [LH.LINDHARD_FP64, LH.LINDHARD_FP32C]
SHAPES = [((16, 8), (1, 1)), ((16, 8), (3, 1)), ((12, 20), (5, 3)), ((10, 9), (1, 3)), ((8, 16), (7, 5)),
          ((128, 4), (11, 1)), ((1040, 5), (1, 1)), ((300, 6), (3, 3))]


def host(t):
    return t.double().cpu().numpy()


def rpa(re, im, V):
    p, b = 1.0 - V * re, V * im
    inv = 1.0 / (p * p + b * b)
    amp = 16 * 2.0 ** -52 * (1.0 + (1.0 + np.abs(V * re)) * (np.abs(p) + np.abs(b)) * inv)
    return im * inv, (re * p - V * im * im) * inv, np.abs(im) * inv * amp, \
        (np.abs(re * p) + np.abs(re) + np.abs(V * im * im)) * inv * amp


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shape,zones", SHAPES)
def test_maps(prec, shape, zones):
    nkx, nky = shape
    zx, zy = zones
    eps = 2.0 ** -23 if prec == LH.LINDHARD_FP32C else 2.0 ** -52
    ulp = lambda x: np.spacing(np.abs(x).astype(np.float32 if prec == LH.LINDHARD_FP32C else np.float64))
    omega = np.array([1, 2, 2.5, 7, 12.25, 20, 31, 40.5, 41, 62, 63]) * (3.0 / 64)
    cfg = dict(eps_table=W.multiband_tables(max(nkx, nky), 1, seed=5)[0][:nky, :nkx].copy(), mu=0.1, nkx=nkx, nky=nky,
               neps=64, emin=-1.5, emax=1.5, gamma=0.07, omega=omega, omega_interp=True, precision=prec, want_rpa=True)
    base = LH.Plan(**cfg)
    plan = LH.Plan(zones=zones, ff_kind=LH.LINDHARD_FF_GAUSS_DX2Y2, ff_width=0.6, **cfg)
    im0, im = base.exec(), plan.exec()
    re0 = base.rpa(0.0)[0]
    one = np.ones((1, nky, nkx))
    m2 = oracle.extend(one, zx, zy, 1, 0.6)[0]
    hx, hy = oracle.zone_axis(nkx, zx)[0], oracle.zone_axis(nky, zy)[0]
    q2 = (2 * np.pi) ** 2 * (np.asarray(hy)[:, None] ** 2 + np.asarray(hx)[None, :] ** 2)
    for got, first in ((im, im0), (plan.rpa(0.7)[0], re0)):
        ref = np.tile(host(first), (1, zy, zx)) * m2
        assert np.all(np.abs(host(got) - ref) <= 2 * eps * np.abs(ref) + 1e-14 * np.abs(host(first)).max())
    for call, V in ((plan.rpa, 0.7), (plan.rpa_coulomb, 0.5)):
        re, imr, rer = call(V)
        at0 = q2 == 0.0
        U = np.full_like(q2, V) if call == plan.rpa else np.where(at0, 0.0, V / np.where(at0, 1.0, q2))
        a, b, da, db = rpa(host(re), host(im), U)
        if call != plan.rpa:
            a[:, at0] = b[:, at0] = 0.0
        assert np.all(np.abs(host(imr) - a) <= ulp(a) + da)
        assert np.all(np.abs(host(rer) - b) <= ulp(b) + db)
        # unaligned and omitted outputs: the same values
        n, st = re.numel(), torch.cuda.current_stream().cuda_stream
        buf = torch.full((n + 3,), 7.0, dtype=re.dtype, device="cuda")
        fn = LH.lindhard_rpa if call == plan.rpa else LH.lindhard_rpa_coulomb
        for pos, full in enumerate((re, imr, rer)):
            ptr = [None, None, None]
            ptr[pos] = buf[1:].data_ptr()
            buf.fill_(7.0)
            fn(plan.handle, V, *ptr, st)
            assert torch.equal(buf[1:n + 1], full.flatten())
            assert torch.all(buf[n + 1:] == 7.0) and buf[0] == 7.0
    out = torch.full((im.numel() + 2,), 7.0, dtype=im.dtype, device="cuda")
    LH.lindhard_exec(plan.handle, out[1:].data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert torch.equal(out[1:-1], im.flatten()) and out[0] == 7.0 and out[-1] == 7.0
    base.close()
    plan.close()
