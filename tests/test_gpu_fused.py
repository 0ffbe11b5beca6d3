"""The cross section in one fused kernel against the path of separate kernels
(which runs while the amplitude kernel is timed): the same points, cuts and
weights, summed in blocks of 256 generated points instead of 64 survivors.
Sums are compensated, so they agree to a few roundings (1e-14); FP64 n = 3 and
4 fused walks add the helicities in the same order.  Histograms are exact sums
of the same weights, scaled from the total: 1e-13 per bin."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu

MODES = {"FIXED_SHAT": dict(sqrt_s=800.0), "UNIFORM_SQRTSHAT": dict(sqrt_shat_lo=200.0, sqrt_shat_hi=1500.0),
         "PP_TOY": dict(sqrt_s=14000.0, sqrt_shat_lo=150.0)}


def _both(H, call):  # noqa: F811
    """(fused, separate) results of call()."""
    fused = call()
    H.timing_enable(True)
    try:
        separate = call()
    finally:
        H.timing_enable(False)
    assert H.timing_read()[1] > 0  # the separate path launched the amplitude kernel
    return fused, separate


def _agree(a, b):
    assert (a["n_gen"], a["n_acc"]) == (b["n_gen"], b["n_acc"])
    for k in ("sigma_fb", "err_fb", "sum_w", "sum_w2"):
        assert abs(a[k] - b[k]) <= 1e-14 * abs(b[k]), (k, a, b)


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("prec", ["FP64", "FP32"])
@pytest.mark.parametrize("n,sampled", [(2, 0), (3, 0), (4, 0), (2, 1), (3, 1), (4, 1), (5, 1)])
def test_fused_equals_separate_kernels(H, n, sampled, prec, mode):  # noqa: F811
    for points in (1, 255, 256, 257, 5003):
        cfg = H.Config(mode=getattr(H, mode), prec=getattr(H, prec), seed=9 + points, npoints=points,
                       helicity_sampling=sampled, **MODES[mode])
        _agree(*_both(H, lambda: H.xsec(n, cfg)))
    for obs, lim in ((H.OBS_PT_MAX, (20.0, 400.0)), (H.OBS_DR_MIN, (0.0, 4.0))):
        (hf, rf), (hs, rs) = _both(H, lambda: H.xsec_hist(n, cfg, obs, 17, *lim))
        _agree(rf, rs)
        assert np.abs(hf - hs).max() <= 1e-13 * rs["sigma_fb"]
        assert abs(hf.sum() / rf["sigma_fb"] - 1) <= 1e-12


@pytest.mark.parametrize("points", [400000, 400001])
def test_both_sides_of_the_fp64_n4_size(H, points):  # noqa: F811
    cfg = H.Config(prec=H.FP64, seed=4, npoints=points, sqrt_s=900.0)
    _agree(*_both(H, lambda: H.xsec(4, cfg)))


def test_chosen_shape_runs_it(H):  # noqa: F811
    """A chosen kernel shape is the one that a cross section runs."""
    cfg = H.Config(prec=H.FP32, seed=6, npoints=30000, sqrt_s=900.0)
    fused = H.xsec(4, cfg)
    try:
        for shape in H.kernel_shapes(4, H.FP32)[:6]:
            H.set_kernel_shape(4, H.FP32, shape)
            got = H.xsec(4, cfg)
            assert got["n_acc"] == fused["n_acc"] and abs(got["sigma_fb"] / fused["sigma_fb"] - 1) <= 1e-5
    finally:
        H.set_kernel_shape(4, H.FP32)


def test_many_bins_and_few(H):  # noqa: F811
    """Histogram bins kept once and four times per workgroup (1024 slots fit four times)."""
    cfg = H.Config(prec=H.FP64, seed=2, npoints=200003, sqrt_s=700.0)
    for bins in (1, 1022, 1023, 4096):
        (hf, rf), (hs, _) = _both(H, lambda: H.xsec_hist(3, cfg, H.OBS_PT_MAX, bins, 20.0, 350.0))
        assert np.abs(hf - hs).max() <= 1e-13 * rf["sigma_fb"]
        assert abs(hf.sum() / rf["sigma_fb"] - 1) <= 1e-12
