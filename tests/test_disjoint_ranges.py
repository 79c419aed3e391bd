"""The set of buffer ranges that keeps the units of one launch apart (CPU).

csrc/disjoint_ranges.h is host code without HIP; tests/disjoint_ranges_check.cpp
drives it beside a list compared pair by pair over 800,000 random groups,
from crowded address spans to sparse ones, touching ends among them.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2412_07210_amd", "csrc")


def test_set_answers_as_a_list_compared_pair_by_pair(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    program = str(tmp_path / "check")
    subprocess.run([cxx, "-O1", "-std=c++17", "-Wall", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", CSRC,
                    os.path.join(HERE, "disjoint_ranges_check.cpp"), "-o", program], check=True)
    r = subprocess.run([program], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    taken, refused = (int(x) for x in r.stdout.split())
    assert taken > 10_000 and refused > 10_000
