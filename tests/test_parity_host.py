"""The recognition of sums of site terms is host code, compiled alone
(tests/parity_host.cpp): with an allocator that fails at each allocation in
turn, and on random operators that are of the form or nearly so."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("parity") / "parity_host")
    csrc = os.path.join(ROOT, "paper_1102_5071_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", csrc,
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "parity_host.cpp"),
                    os.path.join(csrc, "parity.cpp"), "-o", exe], check=True)
    return exe


def test_every_failing_allocation_is_answered(exe):
    run = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr              # nothing terminates
    plain, total, found = map(int, run.stdout.split())
    assert plain == 1 and total > 15 and found < total


@pytest.mark.parametrize("seed", range(4))
def test_a_form_found_gives_the_operator_back(exe, seed):
    run = subprocess.run([exe, str(seed)], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0
    trials, whole, tries, changed = map(int, run.stdout.split())
    assert whole == trials and 0 < changed < tries
