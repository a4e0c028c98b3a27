"""The kernels' own log, exp and expm1 on the CPU against long double (tests/mathcheck/
check_log_exp.cpp): 1.5 units in the last place, the bar of the kernels' sines and cosines --
each is a last rounding, at most half a unit, of terms whose own roundings are below one."""
import json
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_log_exp_expm1_within_one_and_a_half_ulp(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "check")
    subprocess.run([cxx, "-std=c++17", "-O2", "-w", "-I", os.path.join(HERE, "mathcheck", "shim"),
                    "-I", os.path.join(ROOT, "paper_1503_06182_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    "-o", exe, os.path.join(HERE, "mathcheck", "check_log_exp.cpp")], check=True)
    got = json.loads(subprocess.run([exe, "300000"], check=True, capture_output=True, text=True).stdout)
    assert got["log"] <= 1.5 and got["exp"] <= 1.5 and got["expm1"] <= 1.5 and got["limits"], got
    print(got)
