"""heget_me2_frame at the sizes where four waves stop sharing a point's helicity
walks, 256 tiles of 64 points at n = 4 and 512 at n = 5, against the oracle.  Bars:
FP64 1e-12 per point; FP32 median 1e-5, 99.9th percentile 1e-3."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_helas import H, frame_events  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,tiles", [(4, 256), (5, 512)])
@pytest.mark.parametrize("past", [0, 1])
def test_both_sides(H, orc, n, tiles, past):  # noqa: F811
    ev = frame_events(orc, n, 970 + n, 61)
    ref = np.array([orc.me2_frame(n, p) for p in ev])
    count = tiles * 64 + past
    many, want = np.resize(ev, (count, *ev.shape[1:])), np.resize(ref, count)
    assert np.abs(H.me2_frame(many, H.FP64) / want - 1).max() <= 1e-12
    rel = np.abs(H.me2_frame(many, H.FP32) / want - 1)
    assert np.median(rel) <= 1e-5 and np.quantile(rel, 0.999) <= 1e-3
