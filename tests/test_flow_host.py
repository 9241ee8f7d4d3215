"""The flow's host code (flow_api.hip) on the CPU, with stand-ins for the HIP runtime and the kernel
launches (tests/flow_host_check.cpp): when any step of a call that changes the parameters fails, the
packed forms the reading calls use still follow the parameters."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2302_05730_amd", "csrc")


def test_packed_forms_follow_the_parameters(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not shutil.which("g++"):
        pytest.skip("hipcc or g++ not available")
    objs = []
    for src in (os.path.join(CSRC, "flow_api.hip"), os.path.join(ROOT, "tests", "flow_host_check.cpp")):
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        r = subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "--offload-arch=gfx950", "-O1",
                            "-std=c++17", "-fPIC", f"-I{os.path.join(ROOT, 'include')}", f"-I{CSRC}", "-c", src,
                            "-o", obj], capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stderr[-4000:]
        objs.append(obj)
    exe = str(tmp_path / "flow_host_check")
    r = subprocess.run(["g++", *objs, "-o", exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout[-2000:] + r.stderr[-2000:]
