"""|M|^2 at n = 5 on both sides of the size where the default kernel changes
(512 tiles of 64 points: below, a walk that splits into helicity chunks; above,
all 32 configurations in FP32 and eight in FP64 per walk), with a ragged last
tile, against the oracle.  Bars as for every amplitude kernel."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_me2 import H, cut_events  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["FP64", "FP32"])
@pytest.mark.parametrize("count", [512 * 64, 512 * 64 + 1, 1100 * 64 + 17])
def test_n5_default_on_both_sides(H, orc, prec, count):  # noqa: F811
    ev = cut_events(orc, 5, 1100.0, 41, 257)
    ref, _ = orc.me2_batch(ev)
    got = H.me2(np.resize(ev, (count, *ev.shape[1:])), getattr(H, prec))
    rel = np.abs(got / np.resize(ref, count) - 1)
    print(f"{prec} {count} points: max {rel.max():.2e} median {np.median(rel):.2e}", flush=True)
    if prec == "FP64":
        assert rel.max() <= 1e-12
    else:
        assert np.median(rel) <= 1e-5 and np.quantile(rel, 0.999) <= 1e-3
