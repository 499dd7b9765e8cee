"""The fused paths' node sums (rhs and d of a BREAKPOINT, section 3 of the
paper) are rounded to FP64 once: tests/fixed_point.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_totals_are_rounded_once(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "fixed_point")
    subprocess.run([cxx, "-std=gnu++17", "-O2", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_1905_02241_amd", "csrc"), os.path.join(ROOT, "tests", "fixed_point.cpp"),
                    "-o", exe, "-lm"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
