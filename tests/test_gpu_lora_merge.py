"""GPU parity of vnm_lora_merge and the mask refresh (Section 4.3, Eq. 10): bit-exact against the
oracle's fixed-order fp32 merge, and the refreshed mask / compressed triple bit-exact as well."""

import numpy as np
import pytest
import torch

import paper_2410_16135_amd as vnm
import synth_inputs as syn
from oracle import vnm_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _adapter(rng, out, inn, r, amp=0.05):
    return (rng.standard_normal((out, r)) * amp).astype(np.float32), (rng.standard_normal((r, inn)) * amp).astype(np.float32)


@pytest.mark.parametrize("out,inn,r", [(128, 128, 16), (70, 333, 4), (200, 77, 64), (1, 8, 1), (257, 1030, 16), (64, 40, 0)])
def test_merge_bit_exact(out, inn, r):
    rng = np.random.default_rng(out + inn + r)
    W, _ = syn.make_weight_and_input(out, inn, 1, seed=out + r)
    B, A = _adapter(rng, out, inn, r)
    got = vnm.vnm_lora_merge(_dev(W), _dev(B), _dev(A), 2.0).cpu().numpy()
    assert np.array_equal(got.view(np.uint16), orc.lora_merge(W, B, A, 2.0).view(np.uint16))


# whole aligned tiles with 1, 2 and 3 rows of A left over after groups of four, and ranks below four
@pytest.mark.parametrize("out,inn,r", [(128, 128, 1), (128, 128, 3), (136, 264, 5), (128, 128, 6), (128, 128, 7), (2048, 4096, 11)])
def test_merge_of_aligned_tiles_bit_exact(out, inn, r):
    test_merge_bit_exact(out, inn, r)


def test_merge_strided_and_in_place():
    rng = np.random.default_rng(9)
    big = _dev(syn.make_weight_and_input(96, 160, 1, seed=9)[0])
    Wt = big[:, :100]                                   # leading dimension 160, width 100
    W = Wt.cpu().numpy().copy()
    B, A = _adapter(rng, 96, 100, 8)
    want = orc.lora_merge(W, B, A, 1.5)
    vnm.vnm_lora_merge(Wt, _dev(B), _dev(A), 1.5, W_merged=Wt)      # in place
    torch.cuda.synchronize()
    assert np.array_equal(Wt.cpu().numpy().view(np.uint16), want.view(np.uint16))


@pytest.mark.parametrize("with_act", [False, True])
@pytest.mark.parametrize("out,inn,V,M", [(128, 160, 64, 5), (96, 200, 32, 8), (200, 77, 16, 7)])
def test_refreshed_mask_bit_exact(out, inn, V, M, with_act):
    rng = np.random.default_rng(out + M)
    W, _ = syn.make_weight_and_input(out, inn, 1, seed=M)
    B, A = _adapter(rng, out, inn, 16, amp=0.1)
    act = (0.5 + rng.random(inn)).astype(np.float32) if with_act else None
    c = vnm.vnm_refresh_mask(_dev(W), _dev(B), _dev(A), 2.0, V, M, act=None if act is None else _dev(act))
    torch.cuda.synchronize()
    merged, mask = orc.refresh_mask(W, B, A, 2.0, V, M, act)
    assert np.array_equal(c.mask.cpu().numpy(), mask)
    score = None if act is None else orc.importance_ria(merged, act)
    values, meta, colidx, _ = orc.compress(merged, V, M, score=score)
    assert np.array_equal(c.values.cpu().numpy().view(np.uint16), values.reshape(-1).view(np.uint16))
    assert np.array_equal(c.meta.cpu().numpy(), meta.reshape(-1))
    assert np.array_equal(c.colidx.cpu().numpy(), colidx.reshape(-1))
    # Eq. 10: the decompressed weight is (W + BA) (.) M
    assert np.array_equal(vnm.vnm_decompress(c).cpu().numpy().view(np.uint16),
                          orc.masked_dense(merged, mask).view(np.uint16))


# One call for the whole refresh: tiles of 32 rows x 512 columns cut off on both sides, one and two column tiles, row tiles
# beyond one group of 32, an odd number of 32-row blocks, spans of one K step, ranks around the groups of four; weights whose
# column sums pass 2^24 (the division then takes its second correction); and an odd number of columns (single steps).
@pytest.mark.parametrize("out,inn,V,M,r,amp", [(32, 8, 32, 4, 1, 1.0), (33, 520, 32, 16, 3, 1.0), (95, 512, 64, 5, 4, 1.0),
                                               (1100, 24, 128, 8, 7, 1.0), (160, 1032, 32, 5, 16, 1.0), (200, 304, 64, 12, 33, 1.0),
                                               (900, 200, 64, 5, 2, 3.0e6), (64, 1000, 128, 16, 0, 1.0), (70, 1030, 64, 5, 4, 1.0)])
def test_refresh_in_one_call(out, inn, V, M, r, amp):
    rng = np.random.default_rng(out + inn)
    W, _ = syn.make_weight_and_input(out, inn, 1, seed=M)
    W = np.clip(W.astype(np.float32) * amp, -60000.0, 60000.0).astype(np.float16)
    B, A = _adapter(rng, out, inn, r, amp=0.1)
    act = (0.5 + rng.random(inn)).astype(np.float32)
    if amp > 1:
        assert float(np.abs(W.astype(np.float64)).sum(0).max()) > 2.0 ** 24 > float(np.abs(W.astype(np.float64)).sum(1).min())
    c = vnm.vnm_refresh_mask(_dev(W), _dev(B), _dev(A), 2.0, V, M, act=_dev(act))
    torch.cuda.synchronize()
    merged, mask = orc.refresh_mask(W, B, A, 2.0, V, M, act)
    values, meta, colidx, _ = orc.compress(merged, V, M, score=orc.importance_ria(merged, act))
    assert np.array_equal(c.mask.cpu().numpy(), mask)
    assert np.array_equal(c.values.cpu().numpy().view(np.uint16), values.reshape(-1).view(np.uint16))
    assert np.array_equal(c.meta.cpu().numpy(), meta.reshape(-1))
    assert np.array_equal(c.colidx.cpu().numpy(), colidx.reshape(-1))
    # the single steps end in the same matrix-core copy, padding aside: the same product on it
    m = vnm.vnm_lora_merge(_dev(W), _dev(B), _dev(A), 2.0)
    c3 = vnm.vnm_prune_compress_scored(m, vnm.vnm_ria_scores(m, _dev(act)), V, M, want_mask=True)
    if inn % 8 == 0:
        X = torch.ones((40, inn), dtype=torch.float16, device=DEV)
        assert torch.equal(vnm.vnm_spmm(X, c, out_dtype=torch.float32), vnm.vnm_spmm(X, c3, out_dtype=torch.float32))


def _refresh_call(lib, W, B, A, act, V, M, merged, c, ws, scale=2.0, **k):
    """vnm_refresh_mask of the library itself: its status."""
    p = lambda t: 0 if t is None else t.data_ptr()
    r = B.shape[1]
    return lib.vnm_refresh_mask(p(W), W.shape[0], W.shape[1], k.get("ldw", W.stride(0)), p(B), B.stride(0), p(A), A.stride(0), r, scale, p(act),
                                V, 2, M, p(merged), merged.stride(0), p(c.values), p(c.meta), p(c.colidx), p(c.mask), p(c.packed), p(ws),
                                k.get("ws_bytes", ws.numel()), torch.cuda.current_stream().cuda_stream)


def _refresh_buffers(out, inn, V, M):
    import ctypes
    lib = vnm.load_library()
    b = ctypes.c_int64(-1)
    assert lib.vnm_refresh_mask_workspace_bytes(out, inn, V, 2, M, ctypes.byref(b)) == 0
    s = vnm.vnm_query_sizes(out, inn, V, M)
    u8 = lambda n, v=0: torch.full((n,), v, dtype=torch.uint8, device=DEV)
    c = vnm.Compressed(torch.zeros(s.values_elems, dtype=torch.float16, device=DEV), u8(s.meta_bytes), u8(s.colidx_bytes),
                       u8(s.packed_bytes) if s.packed_bytes else None, out, inn, V, M, u8(out * inn, 7).view(out, inn))
    return lib, c, u8(max(b.value, 1), 255), b.value


def _three_calls(W, B, A, act, V, M):
    m = vnm.vnm_lora_merge(W, B, A, 2.0)
    c = vnm.vnm_prune_compress_scored(m, vnm.vnm_ria_scores(m, act), V, M, want_mask=True)
    return m, c


def _bits_equal(c, d):
    """The triple and the mask, and the matrix-core copies: packed from the triple, both must decompress and multiply alike."""
    assert torch.equal(c.values.view(torch.int16), d.values.view(torch.int16))
    assert torch.equal(c.meta, d.meta) and torch.equal(c.colidx, d.colidx) and torch.equal(c.mask, d.mask)


def _packed_sections(c):
    """The written parts of the matrix-core copy: three sections, each starting on a 256-byte boundary."""
    up = lambda x: (x + 255) // 256 * 256
    Rp, S = (-(-c.out // c.V) * c.V + 63) // 64, -(-(-(-c.inn // c.M)) // 8)
    parts, off = [], 0
    for nbytes in (Rp * S * 2048, Rp * S * 256, Rp * S * 32 * (2 if c.V == 32 else 1)):
        parts.append(c.packed[off:off + nbytes])
        off += up(nbytes)
    return torch.cat(parts)


# (out, in, V, M, K steps of a workgroup, rows a thread requests at a time): every number of steps and every batch of the pruning
# inside a refresh; at 8 steps more columns than threads.  The rules' own values are checked where they are compiled.
SPANS = [(2400, 2048, 32, 5, 8, 6), (2048, 2048, 64, 5, 4, 6), (1000, 1000, 32, 8, 2, 4), (1280, 2560, 128, 10, 2, 12), (2048, 2000, 128, 8, 2, 8),
         (200, 304, 64, 12, 1, 4), (4096, 1024, 32, 4, 8, 4), (2000, 3000, 64, 8, 4, 8)]


@pytest.mark.parametrize("out,inn,V,M,steps,batch", SPANS)
def test_refresh_is_its_single_calls(out, inn, V, M, steps, batch):
    g = torch.Generator(device=DEV)
    g.manual_seed(out + inn)
    rn = lambda *s: torch.randn(s, generator=g, device=DEV)
    W, B, A = (rn(out, inn) * 0.02).half(), rn(out, 6) * 0.01, rn(6, inn) * 0.05
    act = torch.rand(inn, generator=g, device=DEV) + 0.1
    # zero rows and columns, activations of zero, weights that do not stay finite: what the single calls make of them
    W[::97] = 0
    B[::97] = 0
    W[:, 5::131] = 0
    A[:, 5::131] = 0
    act[3::61] = 0
    W[1::211, 7::113] = float("inf")
    W[2::223, 9::127] = float("nan")
    lib, c, ws, need = _refresh_buffers(out, inn, V, M)
    merged = torch.empty_like(W)
    assert need > 0 and _refresh_call(lib, W, B, A, act, V, M, merged, c, ws) == 0          # (no way round it)
    m, d = _three_calls(W, B, A, act, V, M)
    assert torch.equal(merged.view(torch.int16), m.view(torch.int16))
    _bits_equal(c, d)
    assert torch.equal(_packed_sections(c), _packed_sections(d))


# sums that pass 2^24 in the rows but not in the columns: the division's second correction through the row branch
@pytest.mark.parametrize("out,inn,V,M", [(64, 4096, 32, 8), (40, 8000, 64, 5)])
def test_refresh_with_large_row_sums(out, inn, V, M):
    g = torch.Generator(device=DEV)
    g.manual_seed(inn)
    W = (torch.randn((out, inn), generator=g, device=DEV) * 8000).clamp(-60000, 60000).half()
    B, A = torch.randn((out, 4), generator=g, device=DEV), torch.randn((4, inn), generator=g, device=DEV)
    act = torch.rand(inn, generator=g, device=DEV) + 0.1
    lib, c, ws, _ = _refresh_buffers(out, inn, V, M)
    merged = torch.empty_like(W)
    assert _refresh_call(lib, W, B, A, act, V, M, merged, c, ws) == 0
    s = merged.double().abs()
    assert float(s.sum(1).min()) > 2.0 ** 24 > float(s.sum(0).max())
    m, d = _three_calls(W, B, A, act, V, M)
    assert torch.equal(merged.view(torch.int16), m.view(torch.int16))
    _bits_equal(c, d)


def test_refresh_call_without_mask_or_packed_copy_and_in_place():
    out, inn, V, M = 160, 1032, 32, 5
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    W = (torch.randn((out, inn), generator=g, device=DEV) * 0.02).half()
    B, A = torch.randn((out, 8), generator=g, device=DEV), torch.randn((8, inn), generator=g, device=DEV)
    act = torch.rand(inn, generator=g, device=DEV) + 0.1
    m, d = _three_calls(W, B, A, act, V, M)
    for mask, packed, in_place in ((False, True, False), (True, False, False), (False, False, False), (True, True, True)):
        lib, c, ws, _ = _refresh_buffers(out, inn, V, M)
        untouched, mine = c.mask.clone(), W.clone()
        if not mask:
            c.mask = None
        if not packed:
            c.packed = None
        merged = mine if in_place else torch.empty_like(W)                 # vnm_lora_merge allows W itself
        assert _refresh_call(lib, mine, B, A, act, V, M, merged, c, ws) == 0
        assert torch.equal(merged.view(torch.int16), m.view(torch.int16))
        if not mask:
            c.mask = d.mask
        _bits_equal(c, d)
        if packed:
            assert torch.equal(_packed_sections(c), _packed_sections(d))


def test_refresh_call_errors():
    out, inn, V, M = 96, 104, 32, 4
    W = torch.zeros((out, inn + 8), dtype=torch.float16, device=DEV)
    B, A = torch.zeros((out, 4), device=DEV), torch.zeros((4, inn + 8), device=DEV)
    act = torch.ones(inn + 8, device=DEV)
    lib, c, ws, need = _refresh_buffers(out, inn, V, M)
    merged = torch.empty((out, inn + 8), dtype=torch.float16, device=DEV)
    call = lambda W=W[:, :inn], A=A[:, :inn], act=act[:inn], merged=merged[:, :inn], c=c, ws=ws, V=V, M=M, **k: _refresh_call(
        lib, W, B, A, act, V, M, merged, c, ws, **k)
    assert call() == 0
    assert call(ws_bytes=need - 1) == 5
    # rows that are not 16-byte aligned are left to the single calls
    assert call(W=W[:, 1:inn + 1]) == 3 and call(A=A[:, 1:inn + 1]) == 3 and call(merged=merged[:, 1:inn + 1]) == 3
    assert call(A=torch.zeros((4, inn + 1), device=DEV)[:, :inn]) == 3
    # patterns that it does not take: the query says so too
    for v, m in ((16, 4), (32, 17), (32, 40)):
        import ctypes
        b = ctypes.c_int64(-1)
        assert lib.vnm_refresh_mask_workspace_bytes(out, inn, v, 2, m, ctypes.byref(b)) == 0 and b.value == 0
        assert call(V=v, M=m, c=vnm.Compressed(c.values, c.meta, c.colidx, None, out, inn, v, m, c.mask)) == 3
    # misaligned for any kernel, null pointers, leading dimensions below the width
    assert call(ws=ws[4:]) == 4 and call(ldw=inn - 8) == 2
    for name in ("values", "meta", "colidx"):
        bad = vnm.Compressed(c.values, c.meta, c.colidx, c.packed, out, inn, V, M, c.mask)
        setattr(bad, name, None)
        assert call(c=bad) == 1
    torch.cuda.synchronize()


# in % 8 == 0, but rows of W or of A that are not 16-byte aligned: the binding goes to the single calls, with the outputs it has
@pytest.mark.parametrize("which", ["W base", "W pitch", "A base", "A pitch"])
def test_refresh_of_unaligned_rows(which):
    out, inn, V, M = 200, 304, 64, 5
    rng = np.random.default_rng(len(which))
    Wh, _ = syn.make_weight_and_input(out, inn, 1, seed=M)
    Bh, Ah = _adapter(rng, out, inn, 4, amp=0.1)
    act = (0.5 + rng.random(inn)).astype(np.float32)
    W, A = _dev(Wh), _dev(Ah)
    place = lambda t, off, pitch: torch.zeros((t.shape[0], pitch), dtype=t.dtype, device=DEV)[:, off:off + inn].copy_(t)
    if which[0] == "W":
        W = place(W, 1, inn + 8) if which == "W base" else place(W, 0, inn + 4)
    else:
        A = place(A, 1, inn + 4) if which == "A base" else place(A, 0, inn + 2)
    B, actd = _dev(Bh), _dev(act)
    torch.cuda.synchronize()
    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    c = vnm.vnm_refresh_mask(W, B, A, 2.0, V, M, act=actd)
    # merged weight, triple, copy, mask, two workspaces, scores: each once
    assert torch.cuda.memory_stats()["allocation.all.allocated"] - before <= 9
    merged, mask = orc.refresh_mask(Wh, Bh, Ah, 2.0, V, M, act)
    values, meta, colidx, _ = orc.compress(merged, V, M, score=orc.importance_ria(merged, act))
    assert np.array_equal(c.mask.cpu().numpy(), mask)
    assert np.array_equal(c.values.cpu().numpy().view(np.uint16), values.reshape(-1).view(np.uint16))
    assert np.array_equal(c.meta.cpu().numpy(), meta.reshape(-1)) and np.array_equal(c.colidx.cpu().numpy(), colidx.reshape(-1))


@pytest.mark.parametrize("out,inn,V,M", [(70, 104, 32, 4), (200, 304, 64, 5), (130, 1000, 128, 16), (64, 72, 64, 9)])
def test_mask_at_any_address(out, inn, V, M):
    W, _ = syn.make_weight_and_input(out, inn, 1, seed=M)
    c = vnm.vnm_prune_compress(_dev(W), V, M, want_mask=True)
    want = orc.compress(W, V, M)[3]
    assert np.array_equal(c.mask.cpu().numpy(), want)
    buf = torch.full((out * inn + 64,), 7, dtype=torch.uint8, device=DEV)
    for off in (1, 8, 12):
        buf.fill_(7)
        c.mask = buf[off:off + out * inn].view(out, inn)
        vnm.vnm_prune_compress(_dev(W), V, M, out=c)
        got = buf.cpu().numpy()
        assert np.array_equal(got[off:off + out * inn].reshape(out, inn), want)
        assert (got[:off] == 7).all() and (got[off + out * inn:] == 7).all()      # nothing around it is touched


def test_merge_llama_shaped_layer_full_size():
    layer = syn.config_llama2_7b()[0]
    W, _ = syn.layer_tensors(layer, tokens=1)
    rng = np.random.default_rng(16)
    B, A = _adapter(rng, layer.out, layer.inn, 16, amp=0.02)
    got = vnm.vnm_lora_merge(_dev(W), _dev(B), _dev(A), 2.0).cpu().numpy()
    assert np.array_equal(got.view(np.uint16), orc.lora_merge(W, B, A, 2.0).view(np.uint16))


def test_merge_argument_errors():
    lib = vnm.load_library()
    W = torch.zeros((8, 16), dtype=torch.float16, device=DEV)
    B = torch.zeros((8, 4), dtype=torch.float32, device=DEV)
    A = torch.zeros((4, 16), dtype=torch.float32, device=DEV)
    call = lambda **k: lib.vnm_lora_merge(k.get("W", W.data_ptr()), 8, 16, k.get("ldw", 16), B.data_ptr(), k.get("ldb", 4),
                                          A.data_ptr(), 16, k.get("r", 4), 2.0, W.data_ptr(), 16, None)
    assert call() == 0
    assert call(W=None) == 1 and call(ldw=8) == 2 and call(ldb=2) == 2 and call(r=-1) == 2
    torch.cuda.synchronize()
