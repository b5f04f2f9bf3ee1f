"""No attention kernel keeps registers in scratch memory: a launch would have the runtime allocate it (the engine promises calls
without device allocation), and its loops would pay for the traffic. Read from the compiler's resource report."""
import os
import re
import subprocess

import pytest

from paper_2509_21841_amd import build

REPORT = ["--cuda-device-only", "-S", "-o", os.devnull, "-Rpass-analysis=kernel-resource-usage"]


@pytest.mark.parametrize("source", ["attn_fwd.hip", "attn_bwd.hip"])
def test_no_scratch(source):
    r = subprocess.run([build._hipcc(), *build.FLAGS, *REPORT, os.path.join(build.CSRC, source)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)]
    assert len(names) == len(scratch) >= 8
    assert not [(n, s) for n, s in zip(names, scratch) if s]
