"""The sizes that the attention kernels are launched with, looked at on the CPU: tests/plans/launch_plans_main.cpp is compiled with
the library's own header and walks capacities up to 2^31 - 1, every number of patterns, long codes and group sizes, with undefined
arithmetic trapped."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2505_06901_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs ROCm's clang++")
def test_launch_plans(tmp_path):
    exe = str(tmp_path / "launch_plans")
    cmd = [CLANG, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
           os.path.join(ROOT, "tests", "plans", "launch_plans_main.cpp"), "-o", exe]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, (run.stdout[-2000:], run.stderr[-2000:])
    assert "conditions hold" in run.stdout
