import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu on the GPU box)")


def load_paper_matrices():
    """Parse tests/golden/paper_matrices.txt -> {(algo, which, field): rows of Fraction}."""
    from fractions import Fraction
    path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "golden", "paper_matrices.txt")
    out, key = {}, None
    for line in open(path):
        line = line.strip()
        if not line or line.startswith("#"):
            continue
        if line.startswith("@"):
            algo, which, field = line[1:].split("|")[0].split()
            key = (algo, which, field)
            out[key] = []
        else:
            out[key].append([Fraction(tok) for tok in line.split()])
    return out


@pytest.fixture(scope="session")
def paper_matrices():
    return load_paper_matrices()


@pytest.fixture(scope="session")
def assembly_file(tmp_path_factory):
    """The library's sources, compiled to assembly."""
    import shutil
    import subprocess
    from paper_2007_12216_amd.build import compile_command
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    path = str(tmp_path_factory.mktemp("isa") / "rnswino.s")
    source = [a for a in compile_command(path) if not a.endswith("plan_math.cpp") and a != "-shared"]
    build = subprocess.run(source + ["-S", "--cuda-device-only"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert build.returncode == 0, build.stdout
    return path


@pytest.fixture(scope="session")
def assembly(assembly_file):
    """{kernel: (instructions, {label: index})}, see test_isa_wait_states.functions."""
    from test_isa_wait_states import functions
    return functions(assembly_file)


@pytest.fixture(scope="session")
def vector_registers(assembly_file):
    """{kernel: vector registers of a wave}, from the assembly's metadata."""
    import re
    found = re.findall(r"\.name:\s+(_Z\w+)(?:(?!\.name:).)*?\.vgpr_count:\s+(\d+)", open(assembly_file).read(), re.S)
    return {name: int(count) for name, count in found}
