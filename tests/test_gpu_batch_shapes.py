"""A batch runs the kernel shapes in use at its call: a repeated batch does not
replay the graph that was captured for other shapes.  On one stream per
configuration a batch's results are those of one call per configuration, to the bit."""
from __future__ import annotations

import pytest

from test_gpu_me2 import H  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [(4, "FP32"), (4, "FP64"), (5, "FP32"), (6, "FP64")])
def test_repeated_batch_follows_a_chosen_shape(H, n, prec):  # noqa: F811
    P = getattr(H, prec)
    cfgs = [H.Config(prec=P, seed=11, npoints=9001, sqrt_s=1000.0), H.Config(prec=P, seed=12, npoints=7003, sqrt_s=1100.0)]
    H.set_batch_schedule(H.BATCH_BRANCHES)
    try:
        before = H.xsec_batch([3, n], cfgs)
        assert before == [H.xsec(3, cfgs[0]), H.xsec(n, cfgs[1])]
        changed = 0
        for shape in H.kernel_shapes(n, P)[:4]:
            H.set_kernel_shape(n, P, shape)
            alone = H.xsec(n, cfgs[1])
            changed += alone != before[1]
            assert H.xsec_batch([3, n], cfgs) == [before[0], alone], shape
        assert changed  # some shape's result differs in its last bits
        H.set_kernel_shape(n, P)
        assert H.xsec_batch([3, n], cfgs) == before
    finally:
        H.set_kernel_shape(n, P)
        H.set_batch_schedule(H.BATCH_AUTO)
