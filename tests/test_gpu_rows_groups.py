"""fc_rows_kernel up to 16 images, four lanes to a row, with several blocks to a workgroup: groups of one, two and four blocks and
what is left of them, rows of no, few and more than sixteen entries side by side, ragged last blocks and block rows."""
import numpy as np
import pytest

import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,bh,bw,d,B", [(4096, 128 * 17, 128, 128, 0.09, 16), (4096, 128 * 26 - 3, 128, 128, 0.04, 9), (4000, 128 * 41, 128, 128, 0.02, 13),
                                           (4096, 128 * 33, 128, 128, 0.30, 16), (2050, 96 * 70 + 1, 100, 96, 0.09, 15), (8192, 64 * 40, 64, 64, 0.15, 16),
                                           (4096, 128 * 9, 128, 128, 0.95, 11)])
def test_groups_of_blocks(M, K, bh, bw, d, B):
    import torch
    rng = np.random.default_rng(M + K)
    # the density varies from row to row: rows of a step differ in length, some have nothing
    keep = rng.random((M, K)) < np.minimum(1.0, d * rng.choice([0.0, 0.3, 1.0, 1.7], (M, 1)))
    L = cl.compress_layer((rng.standard_normal((M, K)) * keep).astype(np.float32), 5, 4, bh, bw, upload=True)
    W = cl.decode_layer(L)[3].cpu().numpy()
    X = np.maximum(rng.standard_normal((B, K)), 0).astype(np.float32)
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
    Y = cl.compressed_fc_forward(L, Xd, bd, relu=True, path=cl.PATH_SPARSE)
    assert torch.equal(Y, cl.compressed_fc_forward(L, Xd, bd, relu=True, path=cl.PATH_SPARSE))
    assert_close(Y.cpu().numpy(), fc_ref(W, X, bias), True)
    L.free()
