"""Registers of kernels whose grid is the workgroups that all compute units hold at
once: one register too many and the last ones run after all others.  The compiler
says what it gave each kernel; nothing runs."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2401_03256_amd import build


@pytest.mark.skipif(not (os.path.exists(build.hipcc()) or shutil.which(build.hipcc())), reason="hipcc not found")
def test_marking_keeps_eight_waves_a_simd():
    # 800 scalar registers a SIMD, 8 waves, 16 of each wave's for the trap
    # handler, given out in sixteens; 512 vector registers
    cmd = [build.hipcc(), *(f for f in build.HIPCC_FLAGS if f != "-shared"), "-I", os.path.join(build.ROOT, "include"),
           "-I", build.CSRC, "--cuda-device-only", "-S", "-o", os.devnull,
           "-Rpass-analysis=kernel-resource-usage", os.path.join(build.CSRC, "rank.hip")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    part = r.stderr.split("k_mark_initial", 1)[1].split("Function Name:", 1)[0]
    use = {k: int(re.search(k + r": (\d+)", part)[1]) for k in ("TotalSGPRs", " VGPRs")}
    assert use["TotalSGPRs"] <= 80 and use[" VGPRs"] <= 64, use
