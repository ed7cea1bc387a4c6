"""The staged product between a few and a few thousand tokens: both numberings of its workgroups over the XCDs,
the K split and its reduction, at the edges of the rules that choose them."""

import pytest
import torch

import paper_2410_16135_amd as vnm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# weight larger than X (tiles of a row group together) and smaller, numbers of workgroups that 8 does not divide,
# exactly 128 (tile, row group) pairs, out not a multiple of 4 (scalar reduction), one token past a tile; short pieces of K;
# 8 and 7 steps unsplit; two pieces in the deep loop at M = 7 and 9; every number of copies per wave
@pytest.mark.parametrize("out,inn,T,V,M", [
    (4096, 1024, 257, 64, 4), (1100, 2048, 385, 64, 4), (640, 4096, 129, 128, 5), (4096, 3840, 1024, 64, 5),
    (1030, 3080, 700, 32, 5), (513, 4096, 300, 64, 8), (2048, 768, 2048, 64, 8), (1026, 8192, 260, 64, 16),
    (520, 2000, 300, 64, 9), (2064, 3000, 900, 128, 9), (520, 2000, 300, 64, 10), (2560, 256, 2049, 64, 4), (2560, 224, 2049, 64, 4),
    (1536, 1024, 2000, 64, 8), (1536, 960, 2000, 64, 8),
    (1536, 3072, 2000, 64, 4), (1536, 3040, 2000, 64, 4), (1536, 5368, 2000, 64, 7), (1536, 7000, 2000, 64, 9)])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
def test_staged_product(out, inn, T, V, M, ydt):
    g = torch.Generator(device=DEV)
    g.manual_seed(out + T)
    c = vnm.vnm_prune_compress((torch.randn((out, inn), generator=g, device=DEV) * 0.02).half(), V, M)
    X = torch.randn((T, inn), generator=g, device=DEV).half()
    Y = vnm.vnm_spmm_staged(vnm.vnm_stage_x(X, M), T, c, out_dtype=ydt)
    W = vnm.vnm_decompress(c).double()
    want, mag = X.double() @ W.t(), X.double().abs() @ W.abs().t()
    # 2 kept products per block, at most 16 K pieces, each addition rounded in fp32; then the rounding of the result
    bound = (2 * -(-inn // M) + 32) * 2.0 ** -24 * mag
    if ydt == torch.float16:
        bound = bound + 2.0 ** -11 * want.abs() + 2.0 ** -24
    assert bool(((Y.double() - want).abs() <= bound).all())


# a split K at the edges of the deep loop: 8 and 7 steps in the last of ten pieces at M = 8, 48 and 47 in the last of two at
# M = 6, its largest M and the next, two column tables; and one step less than a split takes (results of 22 to 78, up to 22)
@pytest.mark.parametrize("out,inn,T,V,M", [
    (2048, 5120, 300, 64, 8), (2048, 5056, 300, 64, 8), (1536, 4608, 2000, 64, 6), (1536, 4560, 2000, 64, 6), (1540, 7200, 900, 64, 9),
    (1540, 7200, 900, 64, 10), (2048, 5000, 700, 32, 5), (1030, 3040, 900, 64, 4), (1030, 3008, 900, 64, 4), (1100, 1920, 500, 64, 8), (1100, 1856, 500, 64, 8)])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
def test_staged_product_split(out, inn, T, V, M, ydt):
    test_staged_product(out, inn, T, V, M, ydt)


# the reduction's epilogue, four results per thread and one: bias and output permutation after the deep loop (M = 8, 9)
# and after the shorter one (two column tables, M = 12), with vector stores and without
@pytest.mark.parametrize("out,inn,T,V,M", [(1536, 1024, 2000, 64, 8), (1540, 1104, 900, 64, 9), (1030, 1024, 900, 64, 8),
                                           (2048, 2048, 700, 32, 5), (1100, 3000, 500, 64, 12), (8192, 1024, 100, 64, 8)])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
@pytest.mark.parametrize("which", [("bias",), ("perm_out",), ("bias", "perm_out")])
def test_staged_product_epilogue(out, inn, T, V, M, ydt, which):
    g = torch.Generator(device=DEV)
    g.manual_seed(out + T)
    c = vnm.vnm_prune_compress((torch.randn((out, inn), generator=g, device=DEV) * 0.02).half(), V, M)
    X = torch.randn((T, inn), generator=g, device=DEV).half()
    kw = {"bias": torch.randn(out, generator=g, device=DEV).half(),
          "perm_out": torch.randperm(out, generator=g, device=DEV).to(torch.int32)}
    kw = {k: v for k, v in kw.items() if k in which}
    Y = vnm.vnm_spmm_fused(X, c, out_dtype=ydt, **kw)
    W = vnm.vnm_decompress(c).double()
    want, mag = X.double() @ W.t(), X.double().abs() @ W.abs().t()
    if "bias" in kw:
        want, mag = want + kw["bias"].double(), mag + kw["bias"].double().abs()
    if "perm_out" in kw:
        po = kw["perm_out"].long()
        want, mag = torch.empty_like(want).index_copy_(1, po, want), torch.empty_like(mag).index_copy_(1, po, mag)
    bound = (2 * -(-inn // M) + 32) * 2.0 ** -24 * mag
    if ydt == torch.float16:
        bound = bound + 2.0 ** -11 * want.abs() + 2.0 ** -24
    assert bool(((Y.double() - want).abs() <= bound).all())


# two wave groups on halves of K, unsplit launches of up to 256 workgroups: 8 steps (4 each), 9 and other odd numbers (one
# group waits a step for the other), every ring (M = 4 to 10), one and two column tables, ragged last row block and token
# tile, 255 and 256 workgroups, boxes of unequal size; 270 workgroups and M = 11 (one group); and eight parts of the token
# tiles (17, 47 and 23 of them, 8 row blocks per workgroup)
KG = [(4096, 320, 1025, 64, 5), (4090, 360, 1100, 64, 5), (2056, 1632, 1500, 64, 4), (1100, 3000, 3000, 128, 7), (2050, 2040, 1300, 64, 6),
      (4096, 1024, 2048, 32, 8), (4104, 1600, 1920, 32, 10), (5504, 680, 1000, 64, 9), (1000, 3080, 2600, 64, 8), (4360, 600, 1920, 64, 5),
      (4096, 1408, 1500, 64, 11), (3080, 768, 2100, 64, 4), (2304, 1536, 6000, 64, 8), (5120, 1200, 2900, 32, 5)]


@pytest.mark.parametrize("out,inn,T,V,M", KG)
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
def test_two_wave_groups(out, inn, T, V, M, ydt):
    test_staged_product(out, inn, T, V, M, ydt)


# the same after pieces of K long enough to be split: the deep loop (M = 8, 9) and the shorter one
@pytest.mark.parametrize("out,inn,T,V,M", [(1030, 8192, 900, 64, 8), (1540, 7200, 900, 64, 9), (2048, 5000, 700, 32, 5), (8192, 3000, 100, 64, 8)])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
@pytest.mark.parametrize("which", [("bias",), ("perm_out",), ("bias", "perm_out")])
def test_split_epilogue(out, inn, T, V, M, ydt, which):
    test_staged_product_epilogue(out, inn, T, V, M, ydt, which)


@pytest.mark.parametrize("out,inn,T,V,M", [(2050, 2040, 1300, 64, 5), (4096, 2048, 2048, 32, 8), (2100, 1500 // 8 * 8, 2900, 64, 8)])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
@pytest.mark.parametrize("which", [("bias",), ("perm_out",), ("bias", "perm_out")])
def test_two_wave_groups_epilogue(out, inn, T, V, M, ydt, which):
    test_staged_product_epilogue(out, inn, T, V, M, ydt, which)


# two wave groups numbered by columns: 49 tiles x 5 groups and 11 x 22, where no box of workgroups fits an XCD
@pytest.mark.parametrize("out,inn,T,V,M", [(1037, 520, 6171, 32, 8), (5400, 520, 1300, 64, 8), (5400, 328, 1300, 128, 5)])
@pytest.mark.parametrize("ydt", [torch.float16, torch.float32])
def test_two_wave_groups_in_columns(out, inn, T, V, M, ydt):
    test_staged_product(out, inn, T, V, M, ydt)
