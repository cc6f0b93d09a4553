"""The input transform's row segments, loaded from multiples of four and shifted into place: every segment of small layers, at every
alignment of the tensor, on the host (csrc/address_math.hpp is compiled into both)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_aligned_row_segments(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "driver")
    cmd = ["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan", "-static-libubsan",
           "-I", os.path.join(ROOT, "paper_2007_12216_amd", "csrc"), os.path.join(ROOT, "tests", "host", "aligned_segments_driver.cpp"), "-o", exe]
    build = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert run.returncode == 0 and "bad=0" in run.stdout, run.stdout[-4000:]
    assert int(run.stdout.split("checks=")[1].split()[0]) > 100000
