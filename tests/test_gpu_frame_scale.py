"""heget_me2_frame over the range of energies a double holds: at n = 2 |M|^2 has no
dimension, so an event in other units has the same one.  Bars: the momenta of the
smallest scale are multiples of 2^-1074, 2^-47 and less of the energies, and a
spinor product divides their rounding by pT / E and its square: 1e-10 with every
pT / E above 0.03 (some 2e-11); 1e-12, the FP64 bar, at the other scales."""
from __future__ import annotations

import numpy as np
import pytest

from test_gpu_helas import H, frame_events  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power,tol", [(1000, 1e-12), (-900, 1e-12), (-1036, 1e-10)])
def test_any_unit_of_energy(H, orc, power, tol):  # noqa: F811
    ev = frame_events(orc, 2, 1000, 60)
    want = H.me2_frame(ev, H.FP64)
    got = H.me2_frame(np.ldexp(ev, power), H.FP64)
    assert np.abs(got / want - 1).max() <= tol
