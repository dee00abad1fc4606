"""The level schedules with the waves, tiles and walk limits of the kernels
(csrc/sweep.hip) on several thousand small graphs, on the host: what a wave
reads before its program runs stays inside the transfer table, and the walk
of sweep_harness.cpp holds (tests/sanitize/sweep_first_record.cpp)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12037_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_first_records_stay_in_the_transfer_table(tmp_path):
    exe = str(tmp_path / "sweep_first_record")
    b = subprocess.run(["g++", "-std=c++17", "-O2", "-D_GLIBCXX_ASSERTIONS", f"-I{ROOT}",
                        os.path.join(ROOT, "tests", "sanitize", "sweep_first_record.cpp"),
                        os.path.join(CSRC, "compile.cpp"), os.path.join(CSRC, "sweep.cpp"),
                        "-o", exe], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    assert "first records ok" in r.stdout
