"""Properties of plans, enumerated on the host with the planner and the arithmetic that it
shares with the kernels."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2111_11581_amd", "csrc")


def _run(name, tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / name)
    subprocess.run([cxx, "-O2", "-std=c++17", "-pthread", "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
                    os.path.join(ROOT, "tests", "native", name + ".cpp"), os.path.join(CSRC, "bsp_plan.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout


def test_no_read_outside_the_input(tmp_path):
    """Loads of 3-wide convs leave the input only in chunks that are loaded element by element."""
    _run("cv_reads", tmp_path)


def test_windows_hold_every_step(tmp_path):
    """No mask that a scheme allows is refused for its kept columns lying far apart."""
    _run("windows", tmp_path)


def test_layers_packed_for_two_kernels(tmp_path):
    """Their plans agree on the tiles and each kernel gets the batches it measured faster at."""
    _run("both", tmp_path)


def test_kept_plans_are_those_of_a_first_call(tmp_path):
    """A thread's kept plans against fresh threads', every pair of layers that differ in one value."""
    _run("reuse", tmp_path)


def test_lists_of_short_block_rows(tmp_path):
    """Lists whose tiles are partly empty are stored with zeros where that measured faster."""
    _run("short_rows", tmp_path)
