"""Kernels that hold their tiles in registers keep nothing in scratch memory, as the compiler reports it.  (No GPU: the source
is compiled for the device alone.)"""
import os
import re
import subprocess

import pytest

from paper_2308_15030_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
@pytest.mark.parametrize("source", ["ffn_split.hip"])
def test_no_scratch(source, tmp_path):
    r = subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-Rpass-analysis=kernel-resource-usage",
                        "-c", os.path.join(build.CSRC, source), "-o", str(tmp_path / "o")], capture_output=True, text=True, check=True)
    report = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+).*?VGPRs Spill: (\d+)", r.stderr, re.S)
    assert report
    for kernel, scratch, spilled in report:
        assert scratch == spilled == "0", kernel
