"""The event kernel's 48-bit digit columns on the CPU (tests/mathcheck/check_fold.cpp): as many
events as the kernel adds between two carries, each with the largest digits, of either sign,
over several stretches, give the integers that 128-bit sums give."""
import json
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_columns_hold_the_largest_digits_between_carries(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "check")
    subprocess.run([cxx, "-std=gnu++17", "-O2", "-w", "-I", os.path.join(HERE, "mathcheck", "shim"),
                    "-I", os.path.join(ROOT, "paper_1503_06182_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    "-o", exe, os.path.join(HERE, "mathcheck", "check_fold.cpp")], check=True)
    got = json.loads(subprocess.run([exe], check=True, capture_output=True, text=True).stdout)
    assert got["sums"] > 0 and got["bad"] == 0, got
