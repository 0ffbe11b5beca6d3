"""Momenta between the kernels of a cross section: where nothing but the
amplitude pass reads them, the two beams are one row, E.  The same points with
all rows kept (a histogram beside them reads the photons') and through the
public generation and amplitude calls give the same weights.

Bars: the amplitude kernel computes the same operations on the same values
either way, so the sums agree to the order in which they are added, 1e-12."""
from __future__ import annotations

import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu


# the kernels that read the short rows: FP64 n = 4 above the fused sizes, n = 5
# (FP32 all configurations per walk and FP64, few and many tiles), n = 6 to 8; at
# a ragged count, and with cuts so tight that the FP64 decision re-reads momenta
@pytest.mark.parametrize("n,prec,points", [(4, "FP64", 400321), (5, "FP32", 70001), (5, "FP64", 1003), (5, "FP64", 70001),
                                           (6, "FP32", 2051), (6, "FP64", 259), (7, "FP32", 515), (8, "FP32", 131)])
@pytest.mark.parametrize("mode", [0, 2])
def test_short_rows_give_the_full_rows_result(H, n, prec, points, mode):  # noqa: F811
    cfg = H.Config(mode=mode, prec=getattr(H, prec), seed=40 + n, npoints=points, sqrt_s=1500.0 if mode == 0 else 14000.0,
                   sqrt_shat_lo=300.0 if mode else 0.0, pt_min=20.0, eta_max=2.5, dr_min=0.4)
    short = H.xsec(n, cfg)
    hist, full = H.xsec_hist(n, cfg, H.OBS_PT_MAX, 10, 0.0, 2000.0)
    assert short["n_acc"] == full["n_acc"] > 0
    for key in ("sum_w", "sum_w2"):
        assert abs(short[key] / full[key] - 1) <= 1e-12, key
