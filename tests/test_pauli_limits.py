"""Pauli-sum plans at their limits, on the host (tests/host/pauli_limits_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("pauli") / "pauli_limits_check")
    csrc = os.path.join(ROOT, "paper_2406_17248_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(ROOT, "tests", "host", "pauli_limits_check.cpp"), os.path.join(csrc, "engine.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("what", ["plan", "coefficients", "grid", "order"])
def test_limits(program, what):
    res = subprocess.run([program, what], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stdout[-2000:] + res.stderr[-2000:]
