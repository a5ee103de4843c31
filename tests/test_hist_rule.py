"""CPU-only: which calls take the direct histogram kernel.  A call that
accumulates into many rows must not (it would read every key once per row to
write the few rows that its flows are in: 440 us instead of 214 for 500 records
on 64,000 rows)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# records, workgroups, windows, rows of a window, accumulate, direct
CASES = [
    (500, 1, 32, 2000, 0, 1), (500, 1, 32, 2000, 1, 0), (2000, 1, 8, 2000, 1, 0), (4000, 1, 1, 8000, 1, 0),
    (4000, 1, 1, 8000, 0, 1), (1000, 1, 1, 2560, 1, 1), (1000, 1, 1, 2562, 1, 0), (1000, 1, 1, 2000, 1, 1),
    (102_400, 25, 1, 128, 1, 1), (102_400, 25, 1, 128, 0, 1), (102_401, 25, 1, 128, 0, 0), (10_000, 2048, 1, 128, 0, 1),
    (10_000, 2049, 1, 128, 0, 0), (16_777, 5, 1, 2000, 0, 1), (16_778, 5, 1, 2000, 0, 0),
]


def test_direct_rule(tmp_path):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("g++ or the HIP headers not installed")
    exe = str(tmp_path / "hist_rule")
    subprocess.check_call(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I", os.path.join(ROOT, "paper_1108_1785_amd", "csrc"),
                           os.path.join(ROOT, "tests", "sanitize", "hist_rule.cpp"), "-o", exe])
    out = subprocess.check_output([exe] + [str(x) for c in CASES for x in c[:5]], text=True).split()
    assert [int(x) for x in out] == [c[5] for c in CASES]
