"""The rounding of the integer path's exact sums of squares
(csrc/logfx_bits.h): it depends on the total alone, not on how the words
that strips and tiles leave split it.  Host only: the header is plain C++
and is compiled here with the system compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sum_of_words_depends_on_the_total_alone(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "exact_sums_check")
    subprocess.run([cxx, "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_1304_3992_amd", "csrc"),
                    os.path.join(ROOT, "tests", "exact_sums_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
