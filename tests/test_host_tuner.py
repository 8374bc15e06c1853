"""The tuner of vector plans times what a solve launches (tests/sanitize/tuner_driver.cpp:
fm_plan.cpp with a host-memory HIP and launches that only record)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2211_07777_amd", "csrc")
ROCM = "/opt/rocm"


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.exists(os.path.join(ROCM, "include", "hip")),
                    reason="needs g++ and the HIP headers")
def test_tuner_times_the_solve_launch(tmp_path):
    exe = str(tmp_path / "tuner_driver")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I" + os.path.join(ROCM, "include"),
                           "-fsanitize=address,undefined", "-fno-sanitize-recover=all", os.path.join(CSRC, "fm_plan.cpp"),
                           os.path.join(HERE, "sanitize", "tuner_driver.cpp"), "-o", exe])
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(res.stdout[-2000:], res.stderr[-4000:])
    assert res.returncode == 0, res.stderr[-4000:]
    assert ", 0 mismatches" in res.stdout
