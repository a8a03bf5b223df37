"""CPU: the library's host side on a stand-in HIP runtime (tests/api_check.cpp):
workspace sizes, and what the launches reach, with no GPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.timeout(300)
def test_host_side_on_a_stand_in_runtime(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "api_check")
    subprocess.run([HIPCC, "-std=c++17", "-O1", "-g", "--offload-arch=gfx950",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-x", "hip",
                    os.path.join(ROOT, "tests", "api_check.cpp"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_1707_08500_amd", "csrc"), "-o", exe],
                   check=True, capture_output=True, timeout=250)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
