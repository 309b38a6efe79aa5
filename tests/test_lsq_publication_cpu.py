"""The one-launch round of the least-squares kernels hands every workgroup's replica to the workgroup that averages them.
A workgroup barrier does not wait for vector stores on gfx950, so each wavefront has to wait for its own before the barrier
that precedes the write-back of the L2: the compiled kernels are read for that wait."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2002_09539_amd import build

HIPCC = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")
def test_every_wavefront_completes_its_stores_before_the_replica_is_published(tmp_path):
    out = str(tmp_path / "lsq.s")
    subprocess.run([HIPCC, *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, "kernels_lsq.hip"), "-o", out],
                   check=True, capture_output=True)
    text = open(out).read()
    kernels = re.findall(r"^(\w*lsq_round\w*kernel\w*):.*?^\s*s_endpgm.*?^\.Lfunc_end", text, re.M | re.S)
    assert len(kernels) == 5, kernels
    for name in kernels:
        lines = text[text.index("\n%s:" % name):].split(".Lfunc_end", 1)[0].splitlines()
        write_back = next(i for i, l in enumerate(lines) if "buffer_wbl2" in l)
        barrier = max(i for i, l in enumerate(lines[:write_back]) if "s_barrier" in l)
        store = max(i for i, l in enumerate(lines[:barrier]) if "global_store" in l)
        assert any(re.search(r"s_waitcnt .*vmcnt\(0\)", l) for l in lines[store:barrier]), name
