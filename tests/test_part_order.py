"""CPU-only build, under UndefinedBehaviorSanitizer, of the order in which the
partition scan takes the classify workgroups (tests/sanitize/part_order_san.cpp):
launches of fewer than 8 workgroups must not divide by the 0 workgroups that
every XCD then has in full."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_partition_order(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers not installed")
    exe = str(tmp_path / "part_order_san")
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_1108_1785_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "part_order_san.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "part_order_san: ok" in r.stdout
