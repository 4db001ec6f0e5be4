"""Compiled kernels (CPU): no scratch memory.  A spilled register of an attention
kernel is reloaded inside its key loop, and each reload waits for every load in
flight, the next stage's among them."""
import os
import re
import subprocess

import pytest

from paper_2609_34325_amd import build


@pytest.mark.parametrize("source", build.SOURCES)
def test_no_scratch(source):
    flags = [f for f in build.HIPCC_FLAGS if f != "-shared"]
    cmd = [build.hipcc(), *flags, "--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
           os.path.join(build.CSRC, source), "-o", os.devnull]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    names = re.findall(r"Function Name: (\S+)", res.stderr)
    scratch = [int(n) for n in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", res.stderr)]
    assert names and len(names) == len(scratch)
    assert not [(n, b) for n, b in zip(names, scratch) if b]
