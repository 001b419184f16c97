"""Launch sizes on the CPU: launch_driver.cpp drives stride_blocks
(paper_2401_03256_amd/csrc/launch.h), which sizes the kernels over an edge list,
built with g++ and AddressSanitizer/UndefinedBehaviorSanitizer."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2401_03256_amd")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_stride_blocks(tmp_path):
    exe = str(tmp_path / "launch")
    subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-Wall", "-Wextra", "-Werror",
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-I", os.path.join(PKG, "csrc"), os.path.join(HERE, "launch_driver.cpp"), "-o", exe],
                   check=True, capture_output=True, text=True, timeout=300)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout + r.stderr[-4000:]
