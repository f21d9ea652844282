"""Launch shapes of the gather sampler's free-running form and of its workgroup
per chain, checked on the CPU against the kernels' LDS layouts and index ranges
(tests/free_plan_check.cpp)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_free_and_few_launch_shapes_stay_in_bounds(tmp_path):
    exe = str(tmp_path / "free_plan_check")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe,
                           os.path.join(HERE, "free_plan_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout[-3000:]
    assert " 0 failures" in out.stdout
