"""The rounds of the batch assembly (csrc/pod_plan.cpp) on the CPU: every cell in
one round, rounds within the scratch that the device has, smaller rounds where
an allocation fails (tests/host_rounds.cpp, g++ with address and undefined
behaviour checks)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2212_14446_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_batch_rounds(tmp_path):
    exe = str(tmp_path / "host_rounds")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-Wall", "-Wextra", "-Werror", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe,
                    os.path.join(ROOT, "tests", "host_rounds.cpp"), os.path.join(CSRC, "pod_plan.cpp")],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout + r.stderr
