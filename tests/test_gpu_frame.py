"""heget_me2_frame on both sides of its split of the helicity walks over waves,
at the edges of its 64-point tiles, and on events with a momentum along an
axis of the given frame.  Bars: the FP64 bar 1e-12 against the oracle, the sum
of two FP64 errors (2e-12) between two evaluations of the same event."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_helas import H, frame_events  # noqa: F401

pytestmark = pytest.mark.gpu

SPLIT_POINTS = 2048 * 64  # from here on one wave takes all walks of a tile


@pytest.mark.parametrize("n", [2, 3, 4, 5])
def test_both_sides_of_the_split_agree(H, orc, n):  # noqa: F811
    ev = frame_events(orc, n, 900 + n, 331)
    many = np.resize(ev, (SPLIT_POINTS + 5, *ev.shape[1:]))
    for prec, tol in ((H.FP64, 2e-12), (H.FP32, 2e-3)):
        one = H.me2_frame(many, prec)
        for count in (1, 63, 65, 331):
            few = H.me2_frame(ev[:count], prec)
            assert np.abs(few / one[:count] - 1).max() <= tol
        assert np.array_equal(one[:331], one[331:662])  # a point's value does not depend on its place


@pytest.mark.parametrize("n", [2, 4])
@pytest.mark.parametrize("which", [0, 1, 2])  # u, ubar, the first photon
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_momentum_along_an_axis(H, orc, n, which, sign):  # noqa: F811
    """Each event turned so that one momentum lies exactly on the +z or -z axis."""
    ev = frame_events(orc, n, 950 + n, 40)
    turned = []
    for p in ev:
        a = sign * p[which, 1:] / np.linalg.norm(p[which, 1:])
        x = np.cross(a, [0.0, 0.6, 0.8])
        x /= np.linalg.norm(x)
        q = p.copy()
        q[:, 1:] = p[:, 1:] @ np.array([x, np.cross(a, x), a]).T
        q[which, 1:3] = 0.0
        q[which, 3] = sign * q[which, 0]
        turned.append(q)
    got = H.me2_frame(np.array(turned), H.FP64)
    ref = np.array([orc.me2_frame(n, p) for p in ev])
    assert np.abs(got / ref - 1).max() <= 2e-12


def test_photon_without_energy_is_flagged(H, orc):  # noqa: F811
    """Every photon needs E > 0: a zero momentum is NaN, alone in its tile."""
    ev = frame_events(orc, 3, 990, 70)
    good = H.me2_frame(ev, H.FP64)
    ev[7, 3] = 0.0
    got, st = H.me2_frame(ev, H.FP64, return_status=True)
    assert st == H.WARN_NONFINITE and not np.isfinite(got[7])
    assert np.array_equal(np.delete(got, 7), np.delete(good, 7))
