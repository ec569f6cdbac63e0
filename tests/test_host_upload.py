"""svo_upload gives back what it holds on the device when host memory runs out
at any of its allocations, on the CPU (tests/host_fuzz/upload_host.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_fuzz", "upload_host.cpp")
HIP_INC = "/opt/rocm/include"


def test_failed_uploads_hold_nothing(tmp_path):
    if not shutil.which("g++") or not os.path.isdir(HIP_INC):
        pytest.skip("g++ or the HIP runtime headers are not available")
    out = str(tmp_path / "upload_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INC,
                    "-I", os.path.join(ROOT, "paper_1911_06001_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    "-Wno-subobject-linkage", SRC, "-o", out],
                   check=True, capture_output=True, text=True, timeout=300)
    p = subprocess.run([out], capture_output=True, text=True, timeout=60)
    assert p.returncode == 0, p.stdout + p.stderr
    assert int(p.stdout.split()[1]) > 10
