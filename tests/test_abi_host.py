"""Host-side checks of the C ABI: the library loads, exports every symbol the header declares, and
rejects bad arguments before touching any device (no GPU needed)."""

import ctypes
import os
import re

import pytest

import paper_2410_16135_amd as vnm
from oracle import vnm_oracle as orc

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    return vnm.load_library()


def test_exports_every_declared_symbol(lib):
    with open(os.path.join(ROOT, "include", "vnm.h")) as f:
        text = f.read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = set(re.findall(r"\b(vnm_[a-z_]+)\s*\(", text))
    assert {"vnm_query_sizes", "vnm_prune_compress", "vnm_pack", "vnm_spmm", "vnm_decompress", "vnm_stage_x",
            "vnm_spmm_staged", "vnm_spmm_workspace_bytes", "vnm_stage_x_bytes", "vnm_spmm_scratch_bytes",
            "vnm_ria_scores", "vnm_prune_compress_scored",
            "vnm_status_string", "vnm_last_hip_error", "vnm_format_version"} <= names
    for n in names:
        assert hasattr(lib, n), n
    assert lib.vnm_format_version() == 1


@pytest.mark.parametrize("out,inn,V,M", [(128, 128, 64, 8), (4096, 4096, 64, 5), (11008, 4096, 128, 7),
                                         (384, 1536, 64, 5), (100, 37, 16, 6), (4096, 11008, 32, 16)])
def test_query_sizes_match_padding_rule(out, inn, V, M):
    s = vnm.vnm_query_sizes(out, inn, V, M)
    out_pad, in_pad, R, B = orc.padded_dims(out, inn, V, M)
    assert (s.out_pad, s.in_pad, s.row_blocks, s.col_blocks) == (out_pad, in_pad, R, B)
    assert s.kc == 4 * B and s.values_elems == out_pad * 2 * B
    assert s.meta_bytes == out_pad * ((B + 1) // 2) and s.colidx_bytes == R * B * 4
    assert (s.packed_bytes > 0) == (V in (32, 64, 128) and M <= 16)
    assert s.packed_bytes % 256 == 0


def test_argument_errors(lib):
    s = vnm.VnmSizes()
    q = lambda *a: lib.vnm_query_sizes(*a, ctypes.byref(s))
    assert q(128, 128, 64, 2, 8) == 0
    assert q(0, 128, 64, 2, 8) == 2 and q(128, -1, 64, 2, 8) == 2            # shape
    assert q(128, 128, 64, 1, 8) == 3 and q(128, 128, 64, 4, 8) == 3         # N must be 2
    assert q(128, 128, 64, 2, 3) == 3 and q(128, 128, 64, 2, 256) == 3       # M range
    assert q(128, 128, 48, 2, 8) == 3 and q(128, 128, 8, 2, 8) == 3          # V set
    assert lib.vnm_query_sizes(128, 128, 64, 2, 8, None) == 1                # null
    # the device entry points validate on the host first: fake non-null pointers are never dereferenced
    P = ctypes.c_void_p
    good = P(0x1000)
    assert lib.vnm_prune_compress(None, 128, 128, 128, 64, 2, 8, good, good, good, None, None, None, 0, None) == 1
    assert lib.vnm_prune_compress(good, 128, 128, 64, 64, 2, 8, good, good, good, None, None, None, 0, None) == 2
    assert lib.vnm_prune_compress(good, 128, 128, 128, 64, 3, 8, good, good, good, None, None, None, 0, None) == 3
    assert lib.vnm_prune_compress(P(0x1001), 128, 128, 128, 64, 2, 8, good, good, good, None, None, None, 0, None) == 4
    assert lib.vnm_prune_compress(good, 128, 128, 128, 64, 2, 8, good, good, good, None, P(0x1010), None, 0, None) == 4
    assert lib.vnm_prune_compress(good, 128, 128, 128, 16, 2, 8, good, good, good, None, good, None, 0, None) == 3
    assert lib.vnm_prune_compress(good, 128, 128, 128, 64, 2, 8, good, good, good, None, None, None, -1, None) == 5
    assert lib.vnm_spmm(None, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None, 0, None) == 1
    assert lib.vnm_spmm(good, -1, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None, 0, None) == 2
    assert lib.vnm_spmm(good, 4, 127, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None, 0, None) == 2
    assert lib.vnm_spmm(good, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 100, 0, 0, None, 0, None) == 2
    assert lib.vnm_spmm(good, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 2, 0, None, 0, None) == 3
    assert lib.vnm_spmm(good, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 9, None, 0, None) == 3
    # forcing the matrix-core path without a packed copy is refused, not silently rerouted
    assert lib.vnm_spmm(good, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 2, None, 0, None) == 3
    # T == 0 is a successful no-op that touches nothing
    assert lib.vnm_spmm(good, 0, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None, 0, None) == 0
    assert lib.vnm_decompress(good, good, good, 128, 128, 64, 2, 8, None, 128, None) == 1
    assert lib.vnm_decompress(good, good, good, 128, 128, 64, 2, 8, good, 5, None) == 2
    assert lib.vnm_pack(good, good, good, 128, 128, 16, 2, 8, good, None) == 3
    assert lib.vnm_pack(good, good, good, 128, 128, 64, 2, 8, P(0x1008), None) == 4
    # the matrix-core kernel needs its workspace: missing or short workspace is an error, not a silent fallback
    a256 = P(0x1000)
    assert lib.vnm_spmm(good, 64, 128, good, good, good, a256, 128, 128, 64, 2, 8, good, 128, 0, 0, None, 0, None) == 5
    assert lib.vnm_spmm(good, 64, 128, good, good, good, a256, 128, 128, 64, 2, 8, good, 128, 0, 0, a256, 16, None) == 5
    b = ctypes.c_int64(-1)
    assert lib.vnm_spmm_workspace_bytes(4096, 4096, 4096, 64, 2, 5, ctypes.byref(b)) == 0 and b.value == (32 * 103 + 3) * 13312
    assert lib.vnm_spmm_workspace_bytes(16, 128, 128, 16, 2, 8, ctypes.byref(b)) == 0 and b.value == 0
    assert lib.vnm_stage_x(good, 4, 100, 128, 5, a256, 1 << 30, None) == 2          # ldx < in
    assert lib.vnm_stage_x(good, 4, 128, 128, 17, a256, 1 << 30, None) == 3         # M beyond the matrix-core range
    assert lib.vnm_stage_x(good, 4, 128, 128, 5, a256, 16, None) == 5
    assert lib.vnm_spmm_staged(a256, 1 << 30, 4, None, 128, 128, 64, 2, 8, good, 128, 0, None, 0, None) == 1
    assert lib.vnm_spmm_staged(a256, 1 << 30, 4, a256, 128, 128, 16, 2, 8, good, 128, 0, None, 0, None) == 3
    assert lib.vnm_spmm_staged(a256, 1 << 30, 4, a256, 128, 128, 64, 2, 8, good, 128, 0, P(0x1008), 1 << 20, None) == 4   # scratch misaligned
    assert lib.vnm_spmm_staged(a256, 1 << 30, 4, a256, 128, 128, 64, 2, 8, good, 128, 0, a256, -1, None) == 5
    # a staged buffer sized for the token tiles alone lacks the three images of slack the product
    # kernel's look-ahead reads: refused on the host (one tile of 128 x 128 at M = 8: 2 images of 20 KiB)
    need = ctypes.c_int64(-1)
    assert lib.vnm_stage_x_bytes(4, 128, 8, ctypes.byref(need)) == 0 and need.value == (2 + 3) * 20480
    assert lib.vnm_spmm_staged(a256, 2 * 20480, 4, a256, 128, 128, 64, 2, 8, good, 128, 0, None, 0, None) == 5
    assert lib.vnm_spmm_staged(a256, need.value - 1, 4, a256, 128, 128, 64, 2, 8, good, 128, 0, None, 0, None) == 5
    assert lib.vnm_spmm_staged(a256, 0, 0, a256, 128, 128, 64, 2, 8, good, 128, 0, None, 0, None) == 0      # T == 0: no-op
    # the entry point without a workspace: same argument errors, and a request beyond its built-in
    # scratch is refused with a message, all before anything touches a device (none exists here)
    assert lib.vnm_spmm_noalloc(None, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None) == 1
    assert lib.vnm_spmm_noalloc(good, 4, 127, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None) == 2
    assert lib.vnm_spmm_noalloc(good, 4, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 2, None) == 3
    assert lib.vnm_spmm_noalloc(good, 0, 128, good, good, good, None, 128, 128, 64, 2, 8, good, 128, 0, 0, None) == 0
    assert lib.vnm_spmm_noalloc(a256, 4200, 4096, good, good, good, a256, 64, 4096, 64, 2, 5, good, 64, 0, 0, None) == 5
    lib.vnm_last_hip_error.restype = ctypes.c_char_p
    assert b"built-in scratch" in lib.vnm_last_hip_error()
    # sizes: staged activations alone, split-K scratch (small token counts only), and their sum
    sb, kb = ctypes.c_int64(-1), ctypes.c_int64(-1)
    assert lib.vnm_stage_x_bytes(4096, 4096, 5, ctypes.byref(sb)) == 0 and sb.value == (32 * 103 + 3) * 13312
    assert lib.vnm_spmm_scratch_bytes(4096, 4096, ctypes.byref(kb)) == 0 and kb.value == 0
    assert lib.vnm_spmm_scratch_bytes(16, 11008, ctypes.byref(kb)) == 0 and kb.value == 16 * 16 * 11008 * 4
    assert lib.vnm_stage_x_bytes(16, 4096, 5, ctypes.byref(sb)) == 0 and sb.value == (103 + 3) * 13312
    assert lib.vnm_spmm_workspace_bytes(16, 11008, 4096, 64, 2, 5, ctypes.byref(b)) == 0 and b.value == sb.value + kb.value
    assert lib.vnm_stage_x_bytes(16, 4096, 17, ctypes.byref(sb)) == 3
    # scores
    assert lib.vnm_ria_scores(None, 8, 8, 8, good, good, 8, good, 128, None) == 1
    assert lib.vnm_ria_scores(good, 8, 8, 4, good, good, 8, good, 128, None) == 2            # ldw < in
    assert lib.vnm_ria_scores(good, 8, 8, 8, good, good, 8, good, 127, None) == 5            # (out + in) * 8 bytes needed
    assert lib.vnm_ria_scores(good, 8, 8, 8, P(0x1002), good, 8, good, 128, None) == 4
    assert lib.vnm_prune_compress_scored(good, None, 128, 128, 128, 128, 64, 2, 8, good, good, good, None, None, None) == 1
    assert lib.vnm_prune_compress_scored(good, good, 128, 128, 128, 100, 64, 2, 8, good, good, good, None, None, None) == 2
    assert lib.vnm_prune_compress_scored(good, good, 128, 128, 128, 128, 64, 3, 8, good, good, good, None, None, None) == 3
    assert lib.vnm_prune_compress_scored(good, P(0x1002), 128, 128, 128, 128, 64, 2, 8, good, good, good, None, None, None) == 4
    assert lib.vnm_status_string(0) == b"ok" and b"null" in lib.vnm_status_string(1)


def test_package_has_no_cpu_fallback():
    """The product package must not import the oracle (nor the oracle the package)."""
    pkg = os.path.join(ROOT, "paper_2410_16135_amd")
    for dirpath, _, files in os.walk(pkg):
        for fn in files:
            if fn.endswith((".py", ".hip", ".h", ".cpp")):
                with open(os.path.join(dirpath, fn)) as f:
                    assert "oracle" not in f.read(), fn
    with open(os.path.join(ROOT, "oracle", "vnm_oracle.py")) as f:
        assert "paper_2410_16135_amd" not in f.read()


def test_bench_refuses_more_than_one_gpu():
    """This build has no distributed path: bench.py --gpus N with N > 1 exits with a message."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                         timeout=120)
    assert res.returncode != 0
    assert "single-GPU" in res.stderr + res.stdout


def test_cached_size_queries_refuse_what_is_no_integer():
    # the answers for equal integers are kept: a float equal to one of them is refused all the same
    c = vnm.Compressed(None, None, None, None, 4096, 4096, 64, 5)
    for query in (lambda T: vnm.vnm_spmm_scratch_bytes(T, 11008), lambda T: vnm.vnm_spmm_workspace_bytes(T, c)):
        assert query(16) > 0
        for T in (16.0, "16", None):
            with pytest.raises((ctypes.ArgumentError, TypeError)):
                query(T)
