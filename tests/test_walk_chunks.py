"""Helicity chunks of walks that keep their top levels outside the unrolled part:
such kernels hold several waves per SIMD, and few tiles are split
over more waves than one for each SIMD.  Read from the bytes that
heget_xsec_device_noalloc says it would need (8 per point and chunk; no GPU)."""
from __future__ import annotations

import ctypes as C
import re

import pytest


def _chunks(H, n, shape, npoints):
    H.set_kernel_shape(n, H.FP32, shape)
    try:
        c = H.Config(prec=H.FP32, seed=1, npoints=npoints, sqrt_s=1000.0).c()
        st = H._lib.heget_xsec_device_noalloc(n, C.byref(c), C.c_void_p(256), None)
        need = int(re.search(r"needs (\d+) bytes", H.last_error()).group(1))
    finally:
        H.set_kernel_shape(n, H.FP32)
    assert st == -2  # HEGET_ERR_RANGE
    # momenta, weight factor, flag, index; block counts and tile sums are less than a byte
    return (need / npoints - (32 * (n + 2) + 8 + 1 + 4)) / 8


@pytest.mark.parametrize("n", [6, 7, 8])
def test_walks_that_hold_several_waves_are_split(n):
    import paper_0908_4403_amd as H
    walks = [s for s in H.kernel_shapes(n, H.FP32) if s[0] < n]
    assert walks
    npoints = 1 << 18  # 2048 tiles of expected survivors
    for s in walks:
        passes = (1 << n) // s[1]
        assert _chunks(H, n, s, npoints) >= min(4, passes), s


def test_unrolled_walks_stay_whole():
    import paper_0908_4403_amd as H
    for s in H.kernel_shapes(5, H.FP32):
        if s[0] == 5:
            assert _chunks(H, 5, s, 1 << 19) < 2, s
