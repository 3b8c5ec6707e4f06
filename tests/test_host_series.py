"""Which plans run their rows in pairs, checked in the plan construction code (CPU
C++): the sides, and how many terms of the deconvolution series each admits."""
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_1409_2014_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no g++")
def test_pairs_follow_the_length_of_the_series(tmp_path):
    exe = tmp_path / "series_driver"
    cmd = ["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", f"-I{ROOT}/include", f"-I{CSRC}", "-I/opt/rocm/include",
           os.path.join(ROOT, "tests", "host", "series_driver.cpp"), os.path.join(CSRC, "plan_host.cpp"),
           "-o", str(exe)]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:]
