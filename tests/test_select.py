"""CPU: the launches that the planner chooses by size (tests/select_check.cpp,
host code only)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.timeout(300)
def test_launches_chosen_by_size(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "select_check")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-g", "--offload-host-only", "-x", "hip",
                    os.path.join(ROOT, "tests", "select_check.cpp"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1707_08500_amd", "csrc"), "-o", exe],
                   check=True, capture_output=True, timeout=200)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
