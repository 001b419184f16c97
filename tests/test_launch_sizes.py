"""Launch sizes on the CPU: launch_driver.cpp drives stride_blocks
(paper_2401_03256_amd/csrc/launch.h), which sizes the kernels over an edge list,
built with g++ and AddressSanitizer/UndefinedBehaviorSanitizer.  And the order of
a load's refusals, which needs no device either: a bad id comes before anything
that the device has to say."""
import os
import shutil
import subprocess

import numpy as np
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


@pytest.mark.skipif(not os.path.exists(os.path.join(PKG, "libdfpr.so")), reason="libdfpr.so not built")
@pytest.mark.parametrize("bad", [-1, 40])
def test_a_bad_id_comes_first(bad):
    from paper_2401_03256_amd import dfpr
    src = np.zeros(3, np.int32)
    dst = np.array([1, bad, 2], np.int32)
    with pytest.raises(dfpr.DfprError) as e:
        dfpr.Graph(40, src, dst)
    assert e.value.code == dfpr.DFPR_E_RANGE and "entry 1" in str(e.value)
