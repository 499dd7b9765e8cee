"""The kernels' FP64 exponentials (mech_math.h) at and beyond the ends of the
range of e^x, on the host: they saturate through the exponent adjust alone."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_exponentials_saturate(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "math_edges")
    subprocess.run([cxx, "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_1905_02241_amd", "csrc"),
                    os.path.join(ROOT, "tests", "math_edges.cpp"), "-o", exe, "-lm"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
