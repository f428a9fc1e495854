"""The planners' worker pool (csrc/qs_pool.h), on the CPU."""

import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2111_02396_amd", "csrc")


def test_loops_of_several_callers_run_at_the_same_time(tmp_path):
    """Six threads' loops cover every index once, and a call that plans does
    not wait until another call's loop has ended."""
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    exe = tmp_path / "pool"
    subprocess.run([cxx, "-O1", "-std=c++17", "-pthread", "-I", CSRC, os.path.join(HERE, "host_pool_probe.cpp"),
                    "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.split()
    assert out == ["wrong", "0", "overlap", "1"]
