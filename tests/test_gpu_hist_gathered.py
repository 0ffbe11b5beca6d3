"""Histograms of survivors whose momenta are gathered from memory (n >= 5, and n >= 6
sampled), with more points than all workgroups take at once, against the same
observable of the event records in numpy.  Bars: bins hold exact sums of the same
weights, 1e-13 of the total, and the weights of points so near an edge (1e-9, some
hundred roundings of the observable) that either side is right."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu


def _observable(k, which):
    pt = np.hypot(k[..., 1], k[..., 2])
    if which == 0:
        return pt.max(axis=1)
    eta, phi = np.arcsinh(k[..., 3] / pt), np.arctan2(k[..., 2], k[..., 1])
    best = np.full(len(k), np.inf)
    for i in range(k.shape[1]):
        for j in range(i):
            dp = np.abs(phi[:, i] - phi[:, j])
            best = np.minimum(best, np.hypot(eta[:, i] - eta[:, j], np.minimum(dp, 2 * np.pi - dp)))
    return best


@pytest.mark.parametrize("n,sampled,points", [(5, 0, 300007), (6, 1, 150001), (7, 1, 140001), (8, 1, 513)])
@pytest.mark.parametrize("which,lo,hi", [(0, 20.0, 300.0), (1, 0.4, 1.2)])
def test_gathered_histogram(H, n, sampled, points, which, lo, hi):  # noqa: F811
    cfg = H.Config(prec=H.FP32, seed=31, npoints=points, sqrt_s=900.0, helicity_sampling=sampled)
    ev = H.xsec_events(n, cfg, momenta=True)
    x, w, bins = _observable(ev["momenta"][:, 2:], which), ev["weight"], 40
    hist, r = H.xsec_hist(n, cfg, which, bins, lo, hi)
    assert r == ev["result"] and r["n_acc"] > 0
    edges = np.linspace(lo, hi, bins + 1)
    at = np.searchsorted(edges, x, side="right")  # 0 below, 1 .. bins, bins + 1 above
    want = np.bincount(at, weights=w, minlength=bins + 2) / points
    near = np.abs(x[:, None] - edges[None, :]) < 1e-9 * hi
    slack = np.array([w[near[:, max(b - 1, 0)] | near[:, min(b, bins)]].sum() for b in range(bins + 2)]) / points
    assert (np.abs(hist - want) <= 1e-13 * r["sigma_fb"] + slack).all()
