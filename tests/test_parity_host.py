"""The recognition of sums of site terms is host code: compiled alone, with an
allocator that fails at each allocation in turn (tests/parity_host.cpp)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_failing_allocation_is_answered(tmp_path):
    exe = str(tmp_path / "parity_host")
    csrc = os.path.join(ROOT, "paper_1102_5071_amd", "csrc")
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I", csrc,
                    "-I", os.path.join(ROOT, "include"), "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "parity_host.cpp"),
                    os.path.join(csrc, "parity.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, run.stderr              # nothing terminates
    plain, total, found = map(int, run.stdout.split())
    assert plain == 1 and total > 40 and found < total
