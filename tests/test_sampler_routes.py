"""Which form of the sampler a call takes, at shapes on both sides of the
measured lines (tests/sampler_routes.cpp, on the CPU)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_sampler_routes(tmp_path):
    exe = str(tmp_path / "sampler_routes")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe,
                           os.path.join(HERE, "sampler_routes.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
