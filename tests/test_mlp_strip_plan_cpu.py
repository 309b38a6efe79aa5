"""The column strips' rule and index arithmetic (csrc/gemm_f32_plan.h, csrc/mlp_strip_plan.h) are plain host code: the host compiler
builds a checker of them."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_mlp_strip import RANGES, SHAPES

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2002_09539_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")


@pytest.fixture(scope="module")
def checker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("strips") / "mlp_strip_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I" + CSRC, os.path.join(HERE, "host_mlp_strip_check.cpp"), "-o", exe], check=True)
    return exe


def test_offsets_of_what_does_not_exist_lie_past_the_operand(checker):
    out = subprocess.run([checker], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert out.stdout.strip().endswith(" 0 mismatches")


def ranges(checker, shapes):
    args = [str(v) for m, dims, batch in shapes for v in (m, batch, dims[1], dims[0])]
    return [int(v) for v in subprocess.run([checker] + args, capture_output=True, text=True, check=True).stdout.split()]


def test_the_parity_tests_reach_the_strips(checker):
    """The shapes of tests/test_gpu_mlp_strip.py take the route that they are listed for."""
    assert ranges(checker, SHAPES) == RANGES
    # and those of its other tests and of test_gpu_dw_layers.py, test_gpu_gemm_split.py
    assert ranges(checker, [(64, (324, 388), 36), (10, (2060, 388), 72), (64, (520, 380), 64), (64, (512, 512), 64), (64, (512, 512), 256)]) == \
        [1, 6, 1, 1, 0]


def test_either_side_of_the_lines(checker):
    took = lambda *q: ranges(checker, [q])[0]   # noqa: E731
    assert took(64, (3072, 1024), 64) == 1 and took(64, (3072, 1024), 128) == 1 and took(64, (3072, 1024), 132) == 0     # samples
    assert took(3, (2488, 1188), 48) == 8 and took(3, (800, 1188), 48) == 0                                             # work
    assert took(19, (748, 1052), 64) == 1 and took(19, (748, 1052), 68) == 0      # 0.54 of a round: enough for up to 64 samples
    assert took(2, (53600, 9996), 32) > 0 and took(2, (53700, 9996), 32) == 0     # 32-bit offsets
