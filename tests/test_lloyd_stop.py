"""The stop of the device codebook training on the CPU: every wave of a launch reads it as the others do, whether the launch's
one writer has been there before it or not (a wave that returned alone would leave its workgroup's barriers)."""
import os
import shutil
import subprocess

import pytest

from .test_sanitizers import ROOT, SAN, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_all_waves_of_a_launch_go_the_same_way(tmp_path):
    exe = str(tmp_path / "lloyd_stop_driver")
    subprocess.check_call(["g++", *SAN, "-std=c++17", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2605_26339_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "lloyd_stop_driver.cpp"), "-o", exe])
    assert "lloyd stop driver ok" in _run(exe)
