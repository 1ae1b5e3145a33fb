"""Kernels that keep a channel's data in registers keep it there: the compiler reports no spills for them."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2102_02344_amd import build


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")
def test_batchnorm_does_not_spill(tmp_path):
    cmd = ["hipcc", *build.FLAGS, "--cuda-device-only", "-c", os.path.join(build.CSRC, "bn.hip"), "-o", str(tmp_path / "bn.o"),
           "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    name, seen, spilled = "", 0, []
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            seen += 1
        m = re.search(r"(VGPRs Spill|ScratchSize \[bytes/lane\]): (\d+)", line)
        if m and int(m.group(2)):
            spilled.append((name, m.group(1), int(m.group(2))))
    assert seen > 0 and not spilled, spilled
