"""The amplitude kernels that spread a point's helicities over the lanes of a
wave (the default from n = 6): against the oracle at the edges of their work
items (1, 2 or 4 points per wave), and against the one-lane-per-point kernels
on enough points that every resident wave walks several items.

Bars: those of every amplitude kernel (FP64 1e-12 per point; FP32 median 1e-5,
99.9th percentile 1e-3); between two FP64 kernels the sum of both, 2e-12."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H, _golden_n8, cut_events  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [6, 7, 8])
@pytest.mark.parametrize("count", [1, 3, 4, 65, 301])
def test_lanes_match_oracle_at_item_edges(H, orc, n, count):  # noqa: F811
    if n == 8:
        ev, ref = _golden_n8(orc, count)
    else:
        ev = cut_events(orc, n, 1200.0, 700 + n, count)
        ref = orc.me2_subsets_batch(ev)[0]
    for prec in (H.FP64, H.FP32):
        assert H.me2_flops(n, prec)[1][7] == 5  # the kernel under test is the one in use
        rel = np.abs(H.me2(ev, prec) / ref - 1)
        print(f"n={n} count={count} prec={prec} max {rel.max():.2e}", flush=True)
        if prec == H.FP64:
            assert rel.max() <= 1e-12
        else:
            assert np.median(rel) <= 1e-5 and np.quantile(rel, 0.999) <= 1e-3


@pytest.mark.parametrize("n,points", [(6, 40961), (7, 20011), (8, 9001)])
def test_lanes_over_several_items_per_wave(H, n, points):  # noqa: F811
    import torch
    mom = torch.empty(((n + 2) * 4, points), dtype=torch.float64, device="cuda")
    w = torch.empty(points, dtype=torch.float64, device="cuda")
    H.gen_points_device(n, 1300.0, mom, w, seed=5)
    mom = mom[:, w > 0].contiguous()
    got = {}
    try:
        for name, shape in (("lanes", None), ("walk", H.kernel_shapes(n, H.FP64)[0])):
            H.set_kernel_shape(n, H.FP64, shape)
            got[name] = torch.zeros(mom.shape[1], dtype=torch.float64, device="cuda")
            H.me2_device(n, mom, got[name], H.FP64)
            torch.cuda.synchronize()
    finally:
        H.set_kernel_shape(n, H.FP64)
    rel = (got["lanes"] / got["walk"] - 1).abs().max().item()
    print(f"n={n} {mom.shape[1]} points: max {rel:.2e}", flush=True)
    assert rel <= 2e-12


@pytest.mark.parametrize("n", [6, 8])
def test_lanes_flag_bad_points(H, orc, n):  # noqa: F811
    """A point off the preconditions is NaN, alone among its wave's points."""
    ev = cut_events(orc, n, 1500.0, 31, 9)
    good = H.me2(ev, H.FP64)
    bad = ev.copy()
    bad[2, 3, 1:3] = 0.0  # a photon along the beam
    bad[6, 0, 1] = 1.0    # a quark off the axis
    got, st = H.me2(bad, H.FP64, return_status=True)
    assert st == H.WARN_NONFINITE and np.isnan(got[[2, 6]]).all()
    keep = np.delete(np.arange(9), [2, 6])
    assert np.array_equal(got[keep], good[keep])
