"""RIA scores at the edges of their launch shapes, bit for bit against the oracle."""

import numpy as np
import pytest
import torch

import paper_2410_16135_amd as vnm
import synth_inputs as syn
from oracle import vnm_oracle as orc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# aligned rows: one pass of the column sums covers 32, 128, 256, 512 or 1024 rows, a workgroup of the scores 1, 4, 8 or 16 --
# numbers of rows one below and above, and no multiples of either; the last two: rows that are not 16-byte aligned
@pytest.mark.parametrize("out,inn", [(1, 64), (31, 72), (33, 72), (127, 304), (200, 1032), (385, 2056), (1000, 200), (1025, 1024), (1535, 1032),
                                     (1537, 264), (3073, 72), (2050, 4104), (3500, 4104), (15, 1031), (1100, 1031)])
def test_ria_scores_at_the_edges_of_the_launch_shapes(out, inn):
    rng = np.random.default_rng(out + inn)
    W, _ = syn.make_weight_and_input(out, inn, 1, seed=out)
    W[-1, :] = 6e-8                                   # the last row counts once: a subnormal, its own row sum
    act = (rng.random(inn) * 4.0 + 0.01).astype(np.float32)
    S = torch.full((out + 1, inn), -1.0, dtype=torch.float32, device=DEV)
    vnm.vnm_ria_scores(torch.from_numpy(W).to(DEV), torch.from_numpy(act).to(DEV), S[:out])
    got = S.cpu().numpy()
    assert np.array_equal(got[:out].view(np.uint32), orc.importance_ria(W, act).view(np.uint32))
    assert bool((got[out] == -1.0).all())             # nothing stored behind the last row


# every span the scored pruning takes (8, 4, 2, 1 K steps of 8 blocks), with steps left over, a ragged last row block
# and a last block that is cut
@pytest.mark.parametrize("out,inn,V,M", [(5470, 592, 32, 4), (3190, 296, 32, 4), (3000, 504, 32, 7), (5753, 328, 64, 8),
                                         (5110, 296, 128, 4), (5000, 248, 32, 16), (200, 304, 64, 5)])
def test_scored_pruning_in_every_span(out, inn, V, M):
    rng = np.random.default_rng(out + M)
    W, _ = syn.make_weight_and_input(out, inn, 1, seed=M)
    S = np.round(rng.random((out, inn)) * 64).astype(np.float32)          # many ties
    c = vnm.vnm_prune_compress_scored(torch.from_numpy(W).to(DEV), torch.from_numpy(S).to(DEV), V, M, want_mask=True)
    torch.cuda.synchronize()
    values, meta, colidx, mask = orc.compress(W, V, M, score=S)
    assert np.array_equal(c.mask.cpu().numpy(), mask)
    assert np.array_equal(c.values.cpu().numpy().view(np.uint16), values.reshape(-1).view(np.uint16))
    assert np.array_equal(c.meta.cpu().numpy(), meta.reshape(-1)) and np.array_equal(c.colidx.cpu().numpy(), colidx.reshape(-1))
    # the matrix-core copy made in the same pass is the one made from the triple
    X = torch.from_numpy(rng.standard_normal((40, inn)).astype(np.float16)).to(DEV)
    again = vnm.vnm_pack(vnm.Compressed(c.values, c.meta, c.colidx, None, out, inn, V, M))
    assert torch.equal(vnm.vnm_spmm(X, c), vnm.vnm_spmm(X, again))
