"""Slabs of plan memory (csrc/plan_memory.h) on a simulated runtime: no piece is handed out while another plan has it or
a launch may still read it, kept plans hold back their own bytes only, little memory is enough, no lock is held in free."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan_memory_on_a_simulated_runtime(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "check")
    subprocess.run([cxx, "-O1", "-g", "-std=c++17", "-Wall", "-Wextra", "-pthread",
                    "-I", os.path.join(ROOT, "paper_2609_26219_amd", "csrc"),
                    os.path.join(ROOT, "tests", "plan_memory_check.cpp"), "-o", exe], check=True)
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr
