"""A tuned n = 5 kernel at other sizes than it was tuned at: the kernels that form
every current once do not split a point's helicities, so after tuning on a large
call a short one still runs what it runs untuned, to the bit."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H, cut_events  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["FP64", "FP32"])
def test_short_calls_keep_their_kernel_after_tuning(H, orc, prec, monkeypatch):  # noqa: F811
    monkeypatch.delenv("HEGET_TUNING_CACHE", raising=False)
    P = getattr(H, prec)
    ev = cut_events(orc, 5, 1000.0, 23, 500)
    ref, _ = orc.me2_batch(ev)
    untuned = H.me2(ev, P)
    cfg = H.Config(prec=P, seed=2, npoints=60001, sqrt_s=1000.0)
    sigma = H.xsec(5, cfg)
    try:
        shape = tuple(H.autotune(5, P, 300000)[k] for k in H.SHAPE_FIELDS)
        assert shape[1] == 32  # a kernel without chunks is the fastest there
        assert np.array_equal(H.me2(ev, P), untuned)
        assert H.xsec(5, cfg) == sigma  # half of 60 001 points expected
        assert H.me2_flops(5, P)[1] == shape
        H.set_kernel_shape(5, P, shape)  # set by the caller: at every size
        forced = H.me2(ev, P)
        assert not np.array_equal(forced, untuned)
        rel = np.abs(forced / ref - 1)
        assert rel.max() <= 1e-12 if prec == "FP64" else np.median(rel) <= 1e-5
    finally:
        H.set_kernel_shape(5, P)
