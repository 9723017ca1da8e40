"""The 3-wide conv kernel's input addresses, enumerated on the host with the planner and the
arithmetic it shares with the kernel: no load leaves the input but those of chunks that are
loaded element by element."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2111_11581_amd", "csrc")


def test_no_read_outside_the_input(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "cv_reads")
    subprocess.run([cxx, "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                    os.path.join(ROOT, "tests", "native", "cv_reads.cpp"), os.path.join(CSRC, "bsp_plan.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
