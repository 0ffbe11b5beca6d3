"""The histogram kernel's last workgroup reads bins that all waves of all
workgroups added to.  A workgroup counts as finished by one thread's release,
which on gfx950 waits for that thread's wave alone, and the barrier before it
waits for no memory operation: so every wave has to wait for its own additions
before the barrier.  Read from the assembly of the kernels (no GPU)."""
from __future__ import annotations

import importlib.util
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _build():
    spec = importlib.util.spec_from_file_location("_heget_build",
                                                  os.path.join(ROOT, "paper_0908_4403_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_every_wave_waits_for_its_additions_before_the_barrier(tmp_path):
    b = _build()
    if not os.path.exists(b.HIPCC):
        pytest.skip("needs hipcc")
    asm = tmp_path / "mc_kernels.s"
    subprocess.run([b.HIPCC, *b.COMMON, "--cuda-device-only", "-S", os.path.join(b.CSRC, "mc_kernels.hip"),
                    "-o", str(asm)], check=True, capture_output=True)
    bodies = re.findall(r"^(_ZN5heget11hist_kernel\w+):[^\n]*\n(.*?)^\.Lfunc_end", asm.read_text(), flags=re.M | re.S)
    assert len(bodies) == 15  # n = 2 .. 8 with two observables, and the fused pass's
    for name, body in bodies:
        code = [line.split(";")[0].strip() for line in body.splitlines()]
        adds = [i for i, c in enumerate(code) if c.startswith("global_atomic_add_x2") and not c.endswith("sc0")]
        assert adds, name
        end = next(i for i in range(adds[-1], len(code)) if code[i] == "s_barrier")
        assert any(re.match(r"s_waitcnt vmcnt\(0\)", c) for c in code[adds[-1]:end]), name
