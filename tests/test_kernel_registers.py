"""What the compiler makes of the kernels: none of them may keep its operands in scratch memory."""

import os
import re
import struct
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


def _kernels_of(library, tmp_path, readelf):
    """{mangled name: bytes of scratch per lane} of the gfx950 code objects in a library built by this package."""
    with open(library, "rb") as f:
        data = f.read()
    magic, at, found = b"__CLANG_OFFLOAD_BUNDLE__", 0, {}
    while (at := data.find(magic, at)) >= 0:
        entries, = struct.unpack_from("<Q", data, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(entries):
            offset, size, length = struct.unpack_from("<QQQ", data, p)
            target = data[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in target and size:
                (tmp_path / "code").write_bytes(data[at + offset:at + offset + size])
                notes = subprocess.run([readelf, "--notes", str(tmp_path / "code")], capture_output=True, text=True, check=True).stdout
                found.update((m.group(1), int(m.group(2))) for m in
                             re.finditer(r"\.name:\s+(_Z\S+).*?\.private_segment_fixed_size: (\d+)", notes, re.S))
        at += len(magic)
    return found


# the same of the built library, for the sources that take minutes to compile: every instantiation of these kernels
@pytest.mark.parametrize("kernel", ["spmm_smfmac_kernel", "spmm_gemv_kernel", "merge_sums_kernel", "ria_prepare_kernel", "prune_pack_kernel",
                                    "retained_kernel", "out_gain_kernel", "spmm_plain_tokens_kernel"])
def test_built_kernels_use_no_scratch_memory(kernel, tmp_path):
    readelf = "/opt/rocm/llvm/bin/llvm-readelf"
    if not os.path.exists(readelf) or build.built_hash() != build.source_hash():
        pytest.skip("llvm-readelf or an up-to-date library not found")
    used = {k: v for k, v in _kernels_of(build.LIB_PATH, tmp_path, readelf).items() if kernel in k}
    assert used, "kernel not found in the library"
    assert {k: v for k, v in used.items() if v} == {}
