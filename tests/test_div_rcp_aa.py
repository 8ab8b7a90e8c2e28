"""The reciprocal-based division of the antialiased weights (div_rcp in the
device header) against the IEEE quotient, for every pair they can produce (a C
program; vectorised, under a second a core)."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("gcc") is None, reason="needs gcc")
def test_div_rcp_equals_ieee_division_for_antialiased_offsets(tmp_path):
    exe = tmp_path / "div_rcp_aa_check"
    subprocess.run(["gcc", "-O3", "-march=native", "-ffp-contract=off", os.path.join(HERE, "div_rcp_aa_check.c"),
                    "-o", str(exe), "-lm"], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout
    assert ", 0 mismatches" in out.stdout
