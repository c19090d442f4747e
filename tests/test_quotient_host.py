"""The quantisation's quotient equals the division for all 2^23 x 2^7 pairs of mantissas (a host program around the
kernel's own function)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_quotient_is_the_division_for_every_mantissa(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    if " fma " not in open("/proc/cpuinfo").read().replace("\n", " "):
        pytest.skip("no fused multiply-add on this CPU")
    exe = str(tmp_path / "quotient_check")
    subprocess.run([gxx, "-O3", "-std=c++17", "-mavx2", "-mfma", "-ffp-contract=off", "-Wall", "-Werror", "-pthread",
                    "-I", os.path.join(ROOT, "paper_2502_14317_amd", "csrc"),
                    os.path.join(ROOT, "tests", "host", "quotient_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout + out.stderr
