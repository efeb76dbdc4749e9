"""Passes over several points: what the program's macros cannot evaluate must
not compile."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2312_07440_amd", "csrc")


@pytest.mark.parametrize("real,points,fine", [("float", 2, True), ("float", 3, False), ("double", 3, True)])
def test_points_of_a_pass(real, points, fine, tmp_path):
    src = tmp_path / "t.cpp"
    src.write_text('#include "mgrw_lorentz.h"\n'
                   f"mgrw::ttk<{real}, {points}> k;\n")
    r = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", CSRC, str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == fine, r.stderr
