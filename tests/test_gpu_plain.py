"""Products on the canonical triple (layers without a matrix-core copy, unaligned rows of X) against the
one-thread-per-output kernel and against fp64."""

import numpy as np
import pytest
import torch

import paper_2410_16135_amd as vnm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _case(out, inn, T, V, M, seed, fused):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    W = (torch.randn((out, inn), generator=g, device=DEV) * 0.02).half()
    X = torch.randn((T, inn), generator=g, device=DEV).half()
    kw = {}
    if fused:
        kw["bias"] = torch.randn(out, generator=g, device=DEV).half()
        kw["perm_in"] = torch.randperm(inn, generator=g, device=DEV).to(torch.int32)
        kw["perm_out"] = torch.randperm(out, generator=g, device=DEV).to(torch.int32)
    return vnm.vnm_prune_compress(W, V, M), X, kw


# tokens: both sides of the switch between the kernels (32), of a token tile (128), of the groups of 4;
# out: remainders of 8 and 16 rows; M above 64 KiB / 260 B per block (one block per chunk) and in < M
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
@pytest.mark.parametrize("out,inn,T,V,M", [
    (1, 3, 1, 16, 4), (17, 33, 2, 16, 5), (100, 1030, 3, 64, 7), (40, 515, 5, 16, 32), (33, 4099, 31, 128, 16),
    (16, 64, 32, 16, 4), (1000, 1030, 333, 16, 7), (70, 129, 127, 16, 255), (250, 77, 129, 32, 200), (64, 20, 128, 16, 17),
    (2049, 101, 257, 64, 6), (4100, 333, 700, 16, 8)])
def test_plain_product(out, inn, T, V, M, ydt, fused):
    c, X, kw = _case(out, inn, T, V, M, out + inn + T, fused)
    call = vnm.vnm_spmm_fused if fused else vnm.vnm_spmm
    Y = call(X, c, out_dtype=ydt, **kw)
    ref = vnm.vnm_spmm_fused(X, c, out_dtype=ydt, path=vnm.PATH_GENERIC, **kw)
    if T >= 32:                                   # the same sums in the same order
        assert torch.equal(Y, ref)
        return
    W64 = vnm.vnm_decompress(c).double()
    Xp = X[:, kw["perm_in"].long()].double() if fused else X.double()
    want, mag = Xp @ W64.t(), Xp.abs() @ W64.abs().t()
    if fused:
        want, mag = want + kw["bias"].double(), mag + kw["bias"].double().abs()
        po = kw["perm_out"].long()
        want, mag = torch.empty_like(want).index_copy_(1, po, want), torch.empty_like(mag).index_copy_(1, po, mag)
    # every sum has at most 2 B + 64 fp32 roundings of partial sums no larger than sum |w x|; then one to the result
    B = -(-inn // M)
    bound = (2 * B + 64) * 2.0 ** -24 * mag
    if ydt == torch.float16:
        bound = bound + 2.0 ** -11 * want.abs() + 2.0 ** -24
    assert bool(((Y.double() - want).abs() <= bound).all())


@pytest.mark.parametrize("T", [1, 7, 40])
def test_plain_infinities_stay_with_the_rows_that_select_them(T):
    c, X, _ = _case(48, 61, T, 16, 5, 9, False)
    # one column of each: a row keeps 2 of the 5 columns of a block, so at most 2 in 5 of them keep either one and
    # the rest are finite (with an infinity in every block no row would be)
    X[:, 7] = float("inf")
    X[0, 23] = float("nan")
    Y = vnm.vnm_spmm(X, c, out_dtype=torch.float32)
    ref = vnm.vnm_spmm(X, c, out_dtype=torch.float32, path=vnm.PATH_GENERIC)
    assert torch.equal(Y.isnan(), ref.isnan()) and torch.equal(Y.isinf(), ref.isinf())
    ok = Y.isfinite()
    assert bool(ok.any()) and torch.allclose(Y[ok], ref[ok], rtol=1e-5, atol=1e-6)


def test_plain_unaligned_rows_of_a_layer_with_a_packed_copy():
    """in is a multiple of 8, but the rows of X start at odd offsets."""
    c, X, _ = _case(128, 160, 50, 64, 5, 3, False)
    wide = torch.zeros((50, 163), dtype=torch.float16, device=DEV)
    wide[:, 1:161] = X
    Y = vnm.vnm_spmm(wide[:, 1:161], c, out_dtype=torch.float32)
    assert torch.equal(Y, vnm.vnm_spmm(X, c, out_dtype=torch.float32, path=vnm.PATH_GENERIC))


# layers with enough column blocks not to go to the scalar kernel: one, two and more tokens by block, and every
# instantiation by token -- 1, 2 and 4 rows per wave with X moved one and two columns at a time, one and several blocks
# per chunk, rows and tokens that fill no tile; more than 2^20 rows
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("out,inn,T,V,M", [
    (17, 64, 1, 16, 4), (18, 129, 2, 16, 5), (33, 127, 4, 32, 9), (40, 4103, 31, 128, 255), (4100, 333, 31, 16, 4),
    (70, 666, 127, 16, 7), (70, 667, 129, 64, 7), (4100, 334, 700, 16, 8), (4100, 333, 700, 16, 8), (11008, 70, 300, 16, 4),
    (11001, 71, 300, 16, 4), (11001, 74, 300, 128, 5), (4100, 2182, 1030, 16, 130), (4100, 2181, 1030, 32, 129),
    (1048577, 62, 33, 16, 4)])
def test_plain_product_in_every_instantiation(out, inn, T, V, M, fused):
    test_plain_product(out, inn, T, V, M, torch.float32, fused)
