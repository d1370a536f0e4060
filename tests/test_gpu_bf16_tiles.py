"""The weight tiles of the bf16 kernel, which its decoders clear while the multipliers are at the next block:
block rows of one block, of a few and of many, so that a split has one, two, an odd and an even number of
them; full tiles followed by nearly empty ones (what is not cleared would show); every image tile."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu

# a product's relative error on the three-product split: the dropped lo x lo term and the two residuals
BF16X3 = 3.0 * 2.0 ** -16


@pytest.mark.parametrize("M", [128, 4096])
@pytest.mark.parametrize("blocks", [1, 2, 3, 4, 7, 20])
@pytest.mark.parametrize("B", [7, 50, 128, 200])
def test_tiles_are_clean(M, blocks, B):
    import torch
    rng = np.random.default_rng(100 * blocks + B)
    K = 128 * blocks - 5
    W = rand_pruned(rng, M, K, 0.01)
    for b in range(0, blocks, 3):
        cols = slice(128 * b, min(128 * b + 128, K))
        W[:, cols] = rand_pruned(rng, M, cols.stop - cols.start, 1.0 if M == 128 else 0.3)
    L = cl.compress_layer(W, 6, 4, 128, 128, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, 6, 4, 128, 128))
    X = rng.standard_normal((B, K)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    Y = cl.compressed_fc_forward(L, Xd, None, relu=False, path=cl.PATH_MFMA_BF16)
    assert_close(Y.cpu().numpy(), fc_ref(oW, X, None), False, product_rel=BF16X3)
    assert torch.equal(Y, cl.compressed_fc_forward(L, Xd, None, relu=False, path=cl.PATH_MFMA_BF16))
    L.free()
