"""What register-blocked plans compute, on the host: their records interpreted as the kernels read
them, against the circuits gate by gate (tests/host/plan_replay.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _host_program(tmp_path, name, *flags, args=()):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / name)
    csrc = os.path.join(ROOT, "paper_2406_17248_amd", "csrc")
    host = os.path.join(ROOT, "tests", "host")
    subprocess.run(["g++", "-std=c++17", *flags, "-I", os.path.join(ROOT, "include"), "-I", csrc, "-I", host,
                    os.path.join(host, name + ".cpp"), os.path.join(csrc, "engine.cpp"), "-o", exe], check=True)
    return subprocess.run([exe, *args], capture_output=True, text=True, timeout=600)


def test_plans_compute_their_circuits(tmp_path):
    """Random and layered circuits of every gate kind on 4 to 12 qubits, both amplitude types, forward
    and reverse with gradients: flips, phase runs, chains, blocks, remaps and their addresses."""
    res = _host_program(tmp_path, "plan_replay", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all")
    assert res.returncode == 0, res.stdout[-3000:] + res.stderr[-3000:]


@pytest.mark.parametrize("gates", ["fixed", "chain"])
def test_rounding_errors_of_plans(tmp_path, gates):
    """Layered circuits in complex128: their plans are no further off than the gates one by one
    (tests/host/plan_accuracy.cpp)."""
    res = _host_program(tmp_path, "plan_accuracy", "-O2", args=(gates,))
    assert res.returncode == 0, res.stdout[-3000:] + res.stderr[-3000:]
