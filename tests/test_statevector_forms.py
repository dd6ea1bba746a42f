"""The rewritten one-qubit unitaries of the state-vector passes lose no
accuracy: their errors against long double are not above those of the
unitaries as given, over circuit depths on both sides of the line from which
they are used (host only: tests/host_sv/replay.cpp replays the kernel's
arithmetic).

Rms errors over 40 circuits of 2^11 to 2^12 outputs scatter by a few percent
(l2) and by about a sixth (the sum, one number a circuit): the bars are 1.1 and
2 times the general form's."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def build(tmp, name, *flags):
    cxx = shutil.which("g++")
    if cxx is None or not os.path.isdir("/opt/rocm/include"):
        pytest.skip("no host C++ compiler or HIP headers")
    exe = str(tmp / name)
    r = subprocess.run([cxx, "-std=c++17", "-D__HIP_PLATFORM_AMD__", *flags,
                        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2205_05836_amd", "csrc"),
                        "-I", "/opt/rocm/include", os.path.join(ROOT, "tests", "host_sv", f"{name}.cpp"), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    return build(tmp_path_factory.mktemp("replay"), "replay", "-O2", "-mfma", "-ffp-contract=off")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return build(tmp_path_factory.mktemp("plan"), "plan", "-O3")


@pytest.mark.parametrize("probs", [0, 1])
@pytest.mark.parametrize("n,layers", [(11, 2), (11, 7), (11, 8), (12, 12), (12, 30)])
def test_errors_are_those_of_general_gates(replay, n, layers, probs):
    r = subprocess.run([replay, str(n), str(layers), "40", str(probs)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    general, rewritten, general_sum, rewritten_sum = map(float, r.stdout.split())
    assert rewritten <= 1.1 * general
    assert rewritten_sum <= 2 * general_sum


@pytest.mark.parametrize("n,layers", [(4, 6), (11, 8), (12, 3), (14, 8), (17, 8), (18, 8), (22, 8), (24, 5), (25, 8),
                                      (30, 8), (34, 3), (18, 200)])
def test_planning_stays_behind_the_passes(plan, n, layers):
    """Every plan is valid, and choosing it costs the host less than half of
    what its passes take by the model (measured: a sixth at 18 qubits, where
    24 shapes took as long as the passes)."""
    r = subprocess.run([plan, str(n), str(layers)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, f"plan check {r.returncode}"
    host, passes = map(float, r.stdout.split())
    assert host < 0.5 * passes
