"""A batch in which a configuration has no points: that one's result is empty, the
others' are those of a batch without it, to the bit, on both schedules."""
from __future__ import annotations

import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["FP64", "FP32"])
@pytest.mark.parametrize("schedule", [1, 2])
@pytest.mark.parametrize("empty", [2, 5, 6])
def test_empty_configuration(H, schedule, empty, prec):  # noqa: F811
    cfg = lambda points: H.Config(prec=getattr(H, prec), seed=1, npoints=points, sqrt_s=1000.0)
    H.set_batch_schedule(schedule)
    try:
        full = H.xsec_batch([3, 5], [cfg(3001), cfg(2003)])
        got = H.xsec_batch([3, empty, 5], [cfg(3001), cfg(0), cfg(2003)])
    finally:
        H.set_batch_schedule(0)
    assert [got[0], got[2]] == full and full[1]["n_acc"] > 0
    assert set(got[1].values()) == {0}
