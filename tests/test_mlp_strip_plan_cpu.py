"""The column strips' index arithmetic (csrc/mlp_strip_plan.h) is plain host code: the host compiler builds a checker of it."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2002_09539_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_offsets_of_what_does_not_exist_lie_past_the_operand(tmp_path):
    exe = str(tmp_path / "mlp_strip_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + CSRC, os.path.join(HERE, "host_mlp_strip_check.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.strip().endswith(" 0 mismatches")
