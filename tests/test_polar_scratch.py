"""The kernels of the polar iteration keep nothing in scratch memory (what the compiler says of them): an address taken
inside their arguments puts a copy of these in every thread's, which half of the launch's time went into."""
import os
import re
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2401_04044_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_no_scratch_memory(tmp_path):
    out = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                          "-packed-fp32-ops", "--offload-device-only", "-Rpass-analysis=kernel-resource-usage", "-c",
                          os.path.join(CSRC, "polar.hip"), "-o", str(tmp_path / "polar.o")], capture_output=True, text=True, check=True).stderr
    found = re.findall(r"Function Name: (\S+).*?ScratchSize \[bytes/lane\]: (\d+)", out, re.S)
    assert len(found) >= 5 and any("poly" in n for n, _ in found), out[-500:]
    assert all(int(size) == 0 for _, size in found), found
