"""The polar encoder's phase cells and its workgroups' shares on the CPU: no conversion of what is no number in range (a pair of
zeros is an ordinary input), and lookup tables only where a workgroup encodes enough to pay for them."""
import os
import shutil
import subprocess

import pytest

from .test_sanitizers import ROOT, SAN, _run


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_cells_and_shares(tmp_path):
    exe = str(tmp_path / "polar_cells_driver")
    subprocess.check_call(["g++", *SAN, "-fsanitize=float-cast-overflow", "-fno-sanitize-recover=float-cast-overflow", "-std=c++17", "-Wall", "-Werror",
                           "-I", os.path.join(ROOT, "paper_2605_26339_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "polar_cells_driver.cpp"), "-o", exe])
    assert "polar cells driver ok" in _run(exe)
