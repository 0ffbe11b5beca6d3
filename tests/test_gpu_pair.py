"""The n = 5 amplitude kernel with two lanes per point: against the oracle at the
edges of its half tiles of 32 points, on both sides of the sizes where it becomes
the default, and with bad points among good ones.  Bars: those of every amplitude
kernel (FP64 1e-12 per point; FP32 median 1e-5, 99.9th percentile 1e-3)."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H, cut_events  # noqa: F401

pytestmark = pytest.mark.gpu


def _within(rel, fp64):
    if fp64:
        assert rel.max() <= 1e-12
    else:
        assert np.median(rel) <= 1e-5 and np.quantile(rel, 0.999) <= 1e-3


@pytest.mark.parametrize("prec,waves", [("FP64", 1), ("FP32", 2)])
@pytest.mark.parametrize("count", [1, 31, 32, 33, 64, 65, 97, 640])
def test_pair_kernel_at_half_tile_edges(H, orc, prec, waves, count):  # noqa: F811
    ev = cut_events(orc, 5, 900.0, 17 + count, count)
    ref, _ = orc.me2_batch(ev)
    try:
        H.set_kernel_shape(5, getattr(H, prec), (5, 32, 2, 1, 0, waves, 1, 6))
        got = H.me2(ev, getattr(H, prec))
    finally:
        H.set_kernel_shape(5, getattr(H, prec))
    rel = np.abs(got / ref - 1)
    print(f"{prec} {count}: max {rel.max():.2e}", flush=True)
    _within(rel, prec == "FP64")


@pytest.mark.parametrize("prec", ["FP64", "FP32"])
@pytest.mark.parametrize("count", [1024 * 64, 1024 * 64 + 1, 4099 * 64 + 33])
def test_n5_default_around_one_wave_per_simd(H, orc, prec, count):  # noqa: F811
    ev = cut_events(orc, 5, 1300.0, 43, 311)
    ref, _ = orc.me2_batch(ev)
    got = H.me2(np.resize(ev, (count, *ev.shape[1:])), getattr(H, prec))
    _within(np.abs(got / np.resize(ref, count) - 1), prec == "FP64")


@pytest.mark.parametrize("prec,waves", [("FP64", 1), ("FP32", 2)])
def test_pair_kernel_flags_bad_points_alone(H, orc, prec, waves):  # noqa: F811
    ev = cut_events(orc, 5, 1000.0, 5, 70)
    ref, _ = orc.me2_batch(ev)
    bad = ev.copy()
    for i in (0, 31, 32, 69):
        bad[i, 3, 0] = -1.0  # a photon with negative energy
    try:
        H.set_kernel_shape(5, getattr(H, prec), (5, 32, 2, 1, 0, waves, 1, 6))
        got = H.me2(bad, getattr(H, prec))
    finally:
        H.set_kernel_shape(5, getattr(H, prec))
    good = np.ones(70, bool)
    good[[0, 31, 32, 69]] = False
    assert np.isnan(got[~good]).all()
    _within(np.abs(got[good] / ref[good] - 1), prec == "FP64")
