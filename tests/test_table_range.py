"""CPU-only build, under UndefinedBehaviorSanitizer, of the layout of a
classify workgroup's range of spilled entries (tests/sanitize/table_range_san.cpp):
sections in bounds, and room for every mix of tiles, so that no shape of a
window sends its entries to device-scope atomics."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_table_range(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers not installed")
    exe = str(tmp_path / "table_range_san")
    subprocess.check_call(["g++", "-std=c++17", "-g", "-O1", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                           "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_1108_1785_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "table_range_san.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
    assert "table_range_san: ok" in r.stdout
