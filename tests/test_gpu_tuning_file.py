"""Tuning files written before the kernels that form every current once existed:
their lines choose among the walks only, and are used where there is nothing but
walks (n <= 4) and not where the default is a kernel they could not choose."""
from __future__ import annotations

import json

import pytest

from test_gpu_me2 import H, cut_events  # noqa: F401

pytestmark = pytest.mark.gpu

KEYS = ("mb", "h", "cl", "wpb", "pf", "wpe", "ppl", "ps")


def test_older_lines(H, orc, tmp_path, monkeypatch):  # noqa: F811
    path = tmp_path / "tune.jsonl"
    monkeypatch.delenv("HEGET_TUNING_CACHE", raising=False)
    ev = {n: cut_events(orc, n, 1500.0, 3, 2) for n in (3, 4, 5, 6)}
    chosen = {n: H.kernel_shapes(n, H.FP32)[2] for n in ev}
    default = {n: H.me2_flops(n, H.FP32)[1] for n in ev}
    line = lambda n, tail: json.dumps({"arch": "gfx950", "prec": H.FP32, "n": n, **dict(zip(KEYS, chosen[n])),
                                       "ms": 0.5, "points": 1048576, **tail}) + "\n"
    path.write_text("".join(line(n, {}) for n in ev))
    monkeypatch.setenv("HEGET_TUNING_CACHE", str(path))
    try:
        H.shutdown()
        H.me2(ev[3], H.FP32)  # the first device use reads the file
        for n in ev:
            assert H.me2_flops(n, H.FP32)[1] == (chosen if n <= 4 else default)[n], n
        # a line of this library's own is used, and keeps the others
        got = H.autotune(4, H.FP32, 4096), H.autotune(6, H.FP32, 4096)
        lines = [json.loads(l) for l in path.read_text().splitlines()]
        assert [l["n"] for l in lines] == [3, 5, 4, 6]
        for n in ev:
            H.set_kernel_shape(n, H.FP32)
        H.shutdown()
        H.me2(ev[3], H.FP32)
        for n, r in zip((4, 6), got):
            assert H.me2_flops(n, H.FP32)[1] == tuple(r[k] for k in H.SHAPE_FIELDS), n
        assert H.me2_flops(3, H.FP32)[1] == chosen[3] and H.me2_flops(5, H.FP32)[1] == default[5]
    finally:
        monkeypatch.delenv("HEGET_TUNING_CACHE")
        for n in ev:
            H.set_kernel_shape(n, H.FP32)
