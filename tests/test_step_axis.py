"""The propagation kernel's step of one axis (csrc/propagate.hip: step_axis)
equals whole-number arithmetic for every distance below 2^16 m, also where the
rate covers it within a minute (rates up to 2^30, beyond the 24 bits of its
product) and where the rate is 0."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_step_axis_is_exact_for_every_rate(tmp_path):
    cc = shutil.which("gcc") or shutil.which("cc")
    if cc is None:
        pytest.skip("no host C compiler")
    exe = tmp_path / "step_axis_check"
    subprocess.run([cc, "-std=c11", "-O2", "-ffp-contract=off", os.path.join(ROOT, "tests", "step_axis_check.c"),
                    "-o", str(exe), "-lm"], check=True)
    n, bad = map(int, subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.split())
    assert n > 15_000_000
    assert bad == 0
