"""Every entry of the slow-tile list is dealt out, on the CPU:
tests/host_fuzz/deal_host.cpp with the trace kernel's own function."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_fuzz", "deal_host.cpp")
HIP_INC = "/opt/rocm/include"


@pytest.mark.parametrize("seed", [1, 2])
def test_every_entry_is_dealt(tmp_path, seed):
    if not shutil.which("g++") or not os.path.isdir(HIP_INC):
        pytest.skip("g++ or the HIP runtime headers are not available")
    out = str(tmp_path / "deal_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INC,
                    "-I", os.path.join(ROOT, "paper_1911_06001_amd", "csrc"),
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all", SRC, "-o", out],
                   check=True, capture_output=True, text=True, timeout=300)
    p = subprocess.run([out, str(seed)], capture_output=True, text=True, timeout=120)
    assert p.returncode == 0, p.stdout + p.stderr
    assert int(p.stdout.split()[-1]) > 0      # sub-lists of different lengths
