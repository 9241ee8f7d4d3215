"""CPU check of the flow-mapped iteration's stratified coordinate (csrc/stratum.h): the same header
compiled for the host against the exact quotient rounded in integers (tests/stratum_check.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_stratum_coordinate_is_the_rounded_quotient(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = tmp_path / "stratum_check"
    subprocess.run([hipcc, "-O2", "-std=c++17", "-ffp-contract=off",
                    f"-I{os.path.join(ROOT, 'paper_2302_05730_amd', 'csrc')}",
                    os.path.join(ROOT, "tests", "stratum_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True, text=True, timeout=300)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout + r.stderr
