"""The batch planner, run on the CPU under the address and undefined-behaviour sanitizers with a
stand-in HIP runtime: every image is placed once, a team's members lie on one XCD before anything that may
queue, and teams keep within the slots they may take."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                    reason="g++ or the HIP headers missing")
def test_batch_plans(tmp_path):
    exe = str(tmp_path / "plan")
    csrc = os.path.join(ROOT, "paper_2410_21207_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                        "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "include"),
                        "-I", csrc, os.path.join(csrc, "sc_api.cpp"), os.path.join(ROOT, "tests", "sanitize", "kernel_stubs.cpp"),
                        os.path.join(ROOT, "tests", "team", "plan.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "all plans hold" in r.stdout, (r.stdout + r.stderr)[-4000:]
