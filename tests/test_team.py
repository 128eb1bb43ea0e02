"""What the workgroups of a team agree on (csrc/sc_team.h), compiled for the host and run there."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(os.path.join(ROCM, "include", "hip")),
                                reason="g++ or the HIP headers missing")


def _run(tmp_path, name, *flags):
    exe = str(tmp_path / name)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-pthread", *flags, "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(ROCM, "include"), "-I", os.path.join(ROOT, "paper_2410_21207_amd", "csrc"),
                        os.path.join(ROOT, "tests", "team", name + ".cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    return r.stdout


def test_every_member_reads_the_same_end_of_a_timed_call(tmp_path):
    assert "all members agreed" in _run(tmp_path, "step_stop")


def test_a_team_is_whoever_has_come(tmp_path):
    assert "all teams formed" in _run(tmp_path, "join")


def test_a_team_is_whoever_has_come_under_a_thread_sanitizer(tmp_path):
    assert "all teams formed" in _run(tmp_path, "join", "-fsanitize=thread")
