"""The index arithmetic of the folded rows' preparation on the host (CPU only).

A layer that is accepted (d <= 65,536, I <= 2^20) can have more than 2^32 16-byte pieces of
folded gate and up rows.  ``tests/host_index/driver.cpp`` walks the pieces with the header that
the kernel and its launch use, at sizes on both sides of 2^32.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


def test_prep_pieces_are_counted_and_walked_beyond_32_bits(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.exists(os.path.join(ROCM, "include", "hip", "hip_runtime.h")):
        pytest.skip("g++ or the HIP headers are not available")
    exe = tmp_path / "index_checks"
    cmd = [gxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__",
           f"-I{ROCM}/include", "-I" + os.path.join(ROOT, "paper_2609_13846_amd", "csrc"),
           os.path.join(ROOT, "tests", "host_index", "driver.cpp"), "-o", str(exe)]
    build = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-4000:]
    assert "index checks passed" in run.stdout
