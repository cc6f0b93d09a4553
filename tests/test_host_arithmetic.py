"""The integer arithmetic that the kernels' addresses and residues rest on, on the host (csrc/address_math.hpp is compiled into both):
divisions by multiplication, the 16-byte row segments at the ends of a tensor, a copy by several workgroups, the size of a staged patch, and the residues of sums
read as binary32 numbers, under AddressSanitizer and UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2007_12216_amd", "csrc")


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("arithmetic") / "address_driver")
    cmd = ["g++", "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-static-libasan", "-static-libubsan",
           "-I", os.path.join(ROOT, "include"), "-I", CSRC, os.path.join(ROOT, "tests", "host", "address_driver.cpp"),
           os.path.join(CSRC, "plan_math.cpp"), "-o", exe]
    build = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout
    return exe


@pytest.mark.parametrize("part", ["divisions", "segments", "copies", "patches", "residues"])
def test_address_and_residue_arithmetic(driver, part):
    run = subprocess.run([driver, part], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert run.returncode == 0 and "bad=0" in run.stdout, run.stdout[-4000:]
    assert int(run.stdout.split("checks=")[1].split()[0]) > 100000
