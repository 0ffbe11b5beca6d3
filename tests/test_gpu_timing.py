"""Timing the amplitude kernel changes no bit of a result: a cross section that
runs as one fused kernel gives that kernel's result with timing on too (the
amplitude kernel runs beside it for its time).  And the fused kernel's weights
against the amplitude kernel's |M|^2 of the same points.

Bars: equality of every bit; for weights against |M|^2 the bars of every
amplitude kernel, once for each of the two."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu

MODES = {"FIXED_SHAT": dict(sqrt_s=800.0), "UNIFORM_SQRTSHAT": dict(sqrt_shat_lo=200.0, sqrt_shat_hi=1500.0),
         "PP_TOY": dict(sqrt_s=14000.0, sqrt_shat_lo=150.0)}


def _timed(H, call):  # noqa: F811
    H.timing_enable(True)
    try:
        return call()
    finally:
        H.timing_enable(False)


@pytest.mark.parametrize("mode", list(MODES))
@pytest.mark.parametrize("prec", ["FP64", "FP32"])
@pytest.mark.parametrize("n,sampled", [(2, 0), (3, 0), (4, 0), (2, 1), (5, 1)])
def test_timed_call_gives_the_same_bits(H, n, sampled, prec, mode):  # noqa: F811
    for points in (1, 257, 70001):
        cfg = H.Config(mode=getattr(H, mode), prec=getattr(H, prec), seed=3 + points, npoints=points,
                       helicity_sampling=sampled, **MODES[mode])
        plain = H.xsec(n, cfg)
        assert _timed(H, lambda: H.xsec(n, cfg)) == plain
    assert H.timing_read()[1] > 0
    args = (n, cfg, H.OBS_PT_MAX, 33, 20.0, 400.0)
    (h0, r0), (h1, r1) = H.xsec_hist(*args), _timed(H, lambda: H.xsec_hist(*args))
    assert r0 == plain and r1 == plain and np.array_equal(h0, h1)
    e0, e1 = H.xsec_events(n, cfg), _timed(H, lambda: H.xsec_events(n, cfg))
    assert np.array_equal(e0["weight"], e1["weight"]) and e0["result"] == e1["result"] == plain


@pytest.mark.parametrize("prec", ["FP64", "FP32"])
def test_calls_without_a_timed_kernel(H, prec):  # noqa: F811
    torch = pytest.importorskip("torch")
    cfg = H.Config(prec=getattr(H, prec), seed=5, npoints=60001, sqrt_s=900.0)
    buf = torch.zeros(64, dtype=torch.uint8, device="cuda")

    def noalloc():
        H.xsec_device_noalloc(4, cfg, buf)
        torch.cuda.synchronize()
        return H.result_from_bytes(buf.cpu().numpy())

    def batch():
        H.set_batch_schedule(2)  # forgets what was captured
        return H.xsec_batch([3, 4], [cfg, cfg])

    try:
        assert _timed(H, noalloc) == noalloc()
        assert _timed(H, batch) == batch()
    finally:
        H.set_batch_schedule(0)


@pytest.mark.parametrize("n", [2, 3, 4])
@pytest.mark.parametrize("prec", ["FP64", "FP32"])
def test_fused_weights_follow_the_amplitude_kernel(H, n, prec):  # noqa: F811
    """At a fixed energy a point's weight is |M|^2 times one constant."""
    cfg = H.Config(prec=getattr(H, prec), seed=8, npoints=5003, sqrt_s=900.0)
    ev = H.xsec_events(n, cfg, momenta=True)
    kept = ev["weight"] > 0
    assert kept.sum() == ev["result"]["n_acc"] > 4000
    ratio = ev["weight"][kept] / H.me2(ev["momenta"][kept], getattr(H, prec))
    rel = np.abs(ratio / np.median(ratio) - 1)
    if prec == "FP64":
        assert rel.max() <= 2e-12
    else:
        assert np.median(rel) <= 2e-5 and np.quantile(rel, 0.999) <= 2e-3
