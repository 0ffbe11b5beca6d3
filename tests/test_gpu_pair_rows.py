"""Cross sections large enough at n = 5 for the kernel with two lanes per point
(more than 65 536 expected survivors): its form that reads one row for the two
beams, with the weights summed in its own epilogue.  Against the form with all rows
(a histogram or event records beside the sums), a walk with one lane per point, and
|M|^2 of the same points.

Bars: the two forms compute the same operations on the same values, 1e-12 between
their sums; between kernels the FP64 bar 1e-12 and in FP32 1e-5 for a sum (the
median bar of a point); per point once the bar of each of the two."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu

WALK = {"FP32": (5, 8, 2, 1, 0, 0, 1, 2), "FP64": (5, 4, 2, 1, 0, 0, 1, 3)}


@pytest.mark.parametrize("prec", ["FP32", "FP64"])
@pytest.mark.parametrize("mode", [0, 2])
def test_two_lane_cross_section(H, prec, mode):  # noqa: F811
    P = getattr(H, prec)
    cfg = H.Config(mode=mode, prec=P, seed=45, npoints=140003, sqrt_s=1500.0 if mode == 0 else 14000.0,
                   sqrt_shat_lo=300.0 if mode else 0.0)
    short = H.xsec(5, cfg)
    assert short["n_acc"] % 32  # a ragged half tile
    _, full = H.xsec_hist(5, cfg, H.OBS_PT_MAX, 10, 0.0, 2000.0)
    ev = H.xsec_events(5, cfg, momenta=mode == 0)
    try:
        H.set_kernel_shape(5, P, WALK[prec])
        walk = H.xsec(5, cfg)
    finally:
        H.set_kernel_shape(5, P)
    assert short["n_acc"] == full["n_acc"] == walk["n_acc"] == (ev["weight"] > 0).sum() > 60000
    for key in ("sum_w", "sum_w2"):
        assert abs(short[key] / full[key] - 1) <= 1e-12, key
        assert abs(short[key] / walk[key] - 1) <= (1e-12 if prec == "FP64" else 1e-5), key
    assert abs(ev["weight"].sum() / short["sum_w"] - 1) <= 1e-12
    if mode == 0:  # a point's weight is |M|^2 times one constant
        kept = np.flatnonzero(ev["weight"] > 0)[:20011]
        ratio = ev["weight"][kept] / H.me2(ev["momenta"][kept], P)
        rel = np.abs(ratio / np.median(ratio) - 1)
        if prec == "FP64":
            assert rel.max() <= 2e-12
        else:
            assert np.median(rel) <= 2e-5 and np.quantile(rel, 0.999) <= 2e-3
