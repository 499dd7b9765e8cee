"""The kernels' FP64 reciprocal and what divides by it (mech_math.h), from a
seed as inexact as the hardware's: tests/math_seeds.cpp."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_one_refinement_is_enough(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "math_seeds")
    subprocess.run([cxx, "-std=gnu++17", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "paper_1905_02241_amd", "csrc"),
                    os.path.join(ROOT, "tests", "math_seeds.cpp"), "-o", exe, "-lm"], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
