"""FP64 |M|^2 at n = 8 is no further from the oracle's stored values than it was in
the walk with one lane per point, which read the events' balance from one end:
median 9.8e-15, 99th percentile 1.37e-13, maximum 2.6e-13 over the 1024 points."""
from __future__ import annotations

import os

import numpy as np
import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "me2_n8_2TeV_seed4_subsets.txt")


def test_n8_errors(H, orc):  # noqa: F811
    rows = [line.split() for line in open(GOLDEN) if line.strip() and not line.startswith("#")]
    ev = np.array([orc.cm_event(8, 2000.0, 4, int(i)) for i, _ in rows])
    ref = np.array([float(v) for _, v in rows])
    assert len(rows) == 1024
    rel = np.abs(H.me2(ev, H.FP64) / ref - 1)
    assert np.median(rel) <= 9.8e-15 and np.quantile(rel, 0.99) <= 1.37e-13 and rel.max() <= 2.6e-13
