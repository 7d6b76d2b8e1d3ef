"""The LDS sizes of a bank's plans hold what the forward kernel lays out in
them, whichever plan the bank ends up with: plain C++, built with g++."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_lds_of_every_plan(tmp_path):
    exe = str(tmp_path / "geometry_driver")
    csrc = os.path.join(ROOT, "paper_1602_05573_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                           os.path.join(csrc, "layout.cpp"), os.path.join(ROOT, "tests", "geometry_driver.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    assert "geometry ok" in r.stdout
