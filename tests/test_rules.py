"""CPU test of the lines between kernels (csrc/sc_rules.h): the assertions of tests/native/rules.cpp hold."""
import os
import subprocess

from paper_2402_07710_amd import build


def test_lines_between_kernels():
    source = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native", "rules.cpp")
    run = subprocess.run([build.CXX, "-std=c++17", "-Wall", "-Werror", "-fsyntax-only", "-I", build.CSRC, source], capture_output=True, text=True)
    assert run.returncode == 0, run.stderr[-3000:]
