"""heget_kernel_shapes names a chosen shape first, also one of the kernels that the
list of walks does not hold (no GPU)."""
from __future__ import annotations

import pytest


@pytest.mark.parametrize("n", range(2, 9))
def test_chosen_shape_leads_the_list(n):
    import paper_0908_4403_amd as H
    for prec in (H.FP32, H.FP64):
        walks = H.kernel_shapes(n, prec)
        used = H.me2_flops(n, prec)[1]
        assert (used in walks) == (n < 5)
        try:
            for shape in (used, walks[-1]):
                H.set_kernel_shape(n, prec, shape)
                listed = H.kernel_shapes(n, prec)
                assert listed[0] == shape == H.me2_flops(n, prec)[1]
                assert sorted(listed) == sorted(walks + [shape] * (shape not in walks))
        finally:
            H.set_kernel_shape(n, prec)
        assert H.kernel_shapes(n, prec) == walks
