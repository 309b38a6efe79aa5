"""The bf16 forward / delta kernel loads its strip of input rows straight into LDS, every wavefront a share of the rows that all of
them read.  A workgroup barrier does not by itself wait for such loads on gfx950, so each wavefront has to wait for its own
before it: the compiled kernels are read for the wait that the source writes out."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2002_09539_amd import build

HIPCC = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_every_wavefront_waits_for_its_rows_before_the_barrier(tmp_path):
    out = str(tmp_path / "conv.s")
    subprocess.run([HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "kernels_conv_bf16.hip"), "-o", out],
                   check=True, capture_output=True)
    bodies = re.findall(r"^(\w*conv3x3_bf16_kernel\w*):(.*?)^\.Lfunc_end", open(out).read(), re.M | re.S)
    assert len(bodies) == 18
    for name, body in bodies:
        lines = [l.strip() for l in body.splitlines()]
        barriers = [i for i, l in enumerate(lines) if l.startswith("s_barrier")]
        assert len(barriers) == 2, name   # the strip has arrived; nobody reads it any more
        first = max(i for i, l in enumerate(lines[:barriers[0]]) if l.startswith(".LBB"))   # the barrier's own basic block
        block = lines[first:barriers[0]]
        wait = max((i for i, l in enumerate(block) if l == "s_waitcnt vmcnt(0)" and "ASMSTART" in block[i - 1]), default=-1)
        assert wait >= 0, name
        assert not any(l.startswith("buffer_load") and l.endswith(" lds") for l in block[wait:]), name
