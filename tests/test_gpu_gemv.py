"""Products of one to four tokens on the vector ALUs: whole and half tiles of the packed copy."""

import pytest
import torch

import paper_2410_16135_amd as vnm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# half tiles with 8 waves and with 16 (a row of X longer than 4096, more than 80 steps), odd and even numbers of K steps, one
# step, fewer pairs of steps than waves, rows that fill no half tile, no tile and no row block, one and two column tables;
# 64 row blocks and 65 (whole tiles)
@pytest.mark.parametrize("T", [1, 2, 3, 4])
@pytest.mark.parametrize("out,inn,V,M", [
    (64, 8, 64, 4), (17, 40, 32, 5), (96, 80, 32, 5), (100, 1032, 64, 8), (130, 3320, 128, 5), (33, 4096, 64, 6), (250, 4104, 64, 16),
    (70, 11008, 32, 7), (4096, 264, 64, 4), (4090, 512, 32, 8), (4097, 264, 64, 4)])
def test_few_tokens(out, inn, V, M, T):
    g = torch.Generator(device=DEV)
    g.manual_seed(out + inn)
    c = vnm.vnm_prune_compress((torch.randn((out, inn), generator=g, device=DEV) * 0.02).half(), V, M)
    X = torch.randn((T, inn), generator=g, device=DEV).half()
    bias = torch.randn(out, generator=g, device=DEV).half()
    po = torch.randperm(out, generator=g, device=DEV).to(torch.int32)
    W = vnm.vnm_decompress(c).double()
    want, mag = X.double() @ W.t(), X.double().abs() @ W.abs().t()
    # 2 kept products per block and at most 64 partial sums, each addition rounded in fp32
    bound = (2 * -(-inn // M) + 64) * 2.0 ** -24 * mag
    Y = vnm.vnm_spmm(X, c, out_dtype=torch.float32)
    assert bool(((Y.double() - want).abs() <= bound).all())
    Z = vnm.vnm_spmm_fused(X, c, bias=bias, perm_out=po, out_dtype=torch.float32)
    want_z = torch.empty_like(want).index_copy_(1, po.long(), want + bias.double())
    bound_z = torch.empty_like(bound).index_copy_(1, po.long(), bound + 2.0 ** -23 * (mag + bias.double().abs()))
    assert bool(((Z.double() - want_z).abs() <= bound_z).all())


# An odd number of K steps leaves half of the last pair of half tiles empty: nothing of it may enter the sums, an infinite weight
# of the first step (whose operand stands in for the missing one) least of all.  One step, three, and one per wave and more.
@pytest.mark.parametrize("T", [1, 2, 4])
@pytest.mark.parametrize("out,steps,V,M", [(64, 1, 64, 4), (40, 3, 32, 8), (128, 17, 64, 5), (64, 33, 128, 8), (200, 101, 64, 5)])
def test_infinite_weight_in_the_first_step(out, steps, V, M, T):
    inn = steps * 8 * M
    g = torch.Generator(device=DEV)
    g.manual_seed(steps)
    c = vnm.vnm_prune_compress((torch.randn((out, inn), generator=g, device=DEV) * 0.02).half(), V, M)
    X = torch.rand((T, inn), generator=g, device=DEV).half() + 0.5               # positive
    finite = vnm.vnm_spmm(X, c, out_dtype=torch.float32)
    c.values.view(-1, 2 * -(-inn // M))[3:out:5, 0] = float("inf")
    vnm.vnm_pack(c)
    Y = vnm.vnm_spmm(X, c, out_dtype=torch.float32)
    assert bool(torch.isposinf(Y[:, 3::5]).all())
    rest = torch.ones(out, dtype=torch.bool, device=DEV)
    rest[3::5] = False
    assert torch.equal(Y[:, rest], finite[:, rest])


# rows of X at the edge of what LDS holds: the widest on half tiles, then whole tiles on 33 row blocks
@pytest.mark.parametrize("out,inn,V,M,T", [(70, 72640, 64, 16, 1), (2080, 72648, 64, 16, 1), (2080, 73664, 32, 16, 1), (2080, 34248, 64, 16, 2),
                                           (2080, 15040, 32, 16, 3), (2080, 15048, 64, 16, 4), (2080, 16064, 64, 12, 4)])
def test_few_tokens_on_wide_layers(out, inn, V, M, T):
    test_few_tokens(out, inn, V, M, T)


# half tiles are dealt out 8 row blocks at a time: 7, 8, 9, 15 and 21 of them, and 63
@pytest.mark.parametrize("T", [1, 4])
@pytest.mark.parametrize("out,inn,V,M", [(448, 264, 64, 4), (512, 264, 32, 4), (550, 520, 64, 8), (960, 264, 128, 5), (1300, 520, 32, 8), (4030, 264, 64, 4)])
def test_order_of_half_tiles(out, inn, V, M, T):
    test_few_tokens(out, inn, V, M, T)
