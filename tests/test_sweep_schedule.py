"""The level schedule of single-spin programs (csrc/sweep.cpp, no HIP) walked
lane by lane on the host with the kernels' index arithmetic: every access in
bounds, every entry written once, the messages, joint weights, marginals and
sums equal to the step-by-step elimination (tests/sanitize/sweep_harness.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12037_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_level_schedule_on_the_host(tmp_path):
    exe = str(tmp_path / "sweep_harness")
    b = subprocess.run(["g++", "-std=c++17", "-O2", "-D_GLIBCXX_ASSERTIONS", f"-I{ROOT}",
                        os.path.join(ROOT, "tests", "sanitize", "sweep_harness.cpp"),
                        os.path.join(CSRC, "compile.cpp"), os.path.join(CSRC, "sweep.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "sweep schedule ok" in r.stdout
