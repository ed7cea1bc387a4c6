"""What the compiler makes of the kernels: none of them may keep its operands in scratch memory."""

import os
import re
import subprocess

import pytest

from paper_2410_16135_amd import build

CSRC = os.path.join(build.PKG_DIR, "csrc")


@pytest.mark.parametrize("source", ["vnm_score.hip", "vnm_spmm_plain.hip", "vnm_prune_fast.hip"])
def test_kernels_use_no_scratch_memory(source, tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    cmd = [hipcc, *build.HIPCC_FLAGS, "-I", os.path.join(build.ROOT, "include"), "--cuda-device-only", "-c",
           os.path.join(CSRC, source), "-o", str(tmp_path / "k.o"), "-Rpass-analysis=kernel-resource-usage"]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert res.returncode == 0, res.stderr[-3000:]
    used = {}
    name = None
    for line in res.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"ScratchSize \[bytes/lane\]: (\d+)", line)
        if m:
            used[name] = int(m.group(1))
    assert used, "no resource report"
    assert {k: v for k, v in used.items() if v} == {}
