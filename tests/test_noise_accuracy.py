"""Accuracy of the kernels' normal draws: their arithmetic (csrc/eco_device.h, compiled for
the CPU with the hardware's reciprocal square root replaced by one that is off by as much
as it may be) against long double, over every 24-bit draw."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2510_18221_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_normals_against_long_double(tmp_path):
    exe = str(tmp_path / "check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-w", "-I" + os.path.join(HERE, "host_hip"), "-I" + CSRC,
                    os.path.join(HERE, "noise_accuracy_check.cpp"), "-o", exe], check=True)
    words = subprocess.run([exe], check=True, capture_output=True, text=True, timeout=300).stdout.split()
    err = {k: float(v) for k, v in zip(words[::2], words[1::2])}
    print(err)
    assert err["one"] == 1               # ln 1 = 0 exactly, and its root next to nothing
    assert err["radius"] <= 1.66         # units of 2^-53, as stated beside the code
    assert err["cossin"] <= 3.0
    assert err["normal"] <= 1.66 + 3.0 + 0.5   # the product's rounding
