"""The rule that says which bands run as rolling blocks, against the steps at which the
kernel takes a block up (host code)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_blocks_are_taken_up_before_their_first_cell(tmp_path):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if not os.path.exists(os.path.join(rocm, "include", "hip", "hip_runtime.h")):
        pytest.skip("HIP headers not found")
    exe = tmp_path / "roll_check"
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2607_06225_amd", "csrc"),
                    os.path.join(ROOT, "tests", "native", "roll_check.cpp"), "-o", str(exe)],
                   check=True, capture_output=True)
    for seed in (1, 2):
        out = subprocess.run([str(exe), str(seed)], capture_output=True, text=True, timeout=300)
        assert out.returncode == 0, out.stdout
        assert int(out.stdout) > 100000
