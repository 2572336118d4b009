"""The tile kernel's requests of X stay inside X whatever the sizes (host arithmetic, see gemm_request_main.cpp)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_requests_outside_x_are_out_of_the_window(tmp_path):
    exe = str(tmp_path / "gemm_request")
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", os.path.join(ROOT, "tests", "gemm_request_main.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "requests in range: ok" in run.stdout, run.stdout
