"""The pinned slots through which waiting calls get their results, on the CPU: a
slot whose kernel was not waited for serves no other call."""
import os
import subprocess

import pytest

from paper_2507_23189_amd import build as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.slow
def test_slots_of_calls_that_failed_stay_taken(tmp_path):
    exe = str(tmp_path / "host_result")
    clang = "/opt/rocm/llvm/bin/clang++"
    if not os.path.exists(clang):
        pytest.skip("clang++ not found")
    subprocess.run([clang, "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include",
                    f"-I{B.INCLUDE}", f"-I{B.CSRC}", os.path.join(ROOT, "tests", "sanitize", "host_result_driver.cpp"),
                    "-o", exe, "-lpthread"], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr
