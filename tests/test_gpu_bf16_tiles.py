"""The weight tiles of the bf16 kernel, which its decoders clear while the multipliers are at the next block:
splits of three to seven blocks, an odd and an even number of them, so that both buffers are used again; in each a full tile
whose buffer the next but one, nearly empty, decodes into (what is not cleared would show); every width of
the image tile.  And layers of one to twenty blocks, most of which have a block or two to a split."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu

# a product's relative error on the three-product split: the dropped lo x lo term and the two residuals
BF16X3 = 3.0 * 2.0 ** -16


# (width of the image tile and splits: the launch shape that 256 CUs give these sizes, which the workspace's size shows)
@pytest.mark.parametrize("M,blocks,B,width,splits", [(2048, 33, 5, 32, 11), (4096, 33, 5, 32, 7), (1024, 33, 129, 64, 9), (2048, 26, 129, 64, 5),
                                                     (4096, 6, 257, 128, 2), (4096, 9, 257, 128, 2), (4096, 14, 257, 128, 2), (4096, 15, 257, 256, 4), (4096, 20, 257, 256, 4)])
def test_tiles_used_again_are_clean(M, blocks, B, width, splits):
    import torch
    rng = np.random.default_rng(blocks + B)
    K = 128 * blocks - 5
    cols = -(-B // width) * width
    assert all(cols != -(-B // w) * w for w in (32, 64, 128, 256) if w != width)
    ends = [blocks * j // splits for j in range(splits + 1)]
    sizes = [b - a for a, b in zip(ends, ends[1:])]
    full = [b % 4 < 2 for b in range(blocks)]                # two full ones, two nearly empty ones: of any two that share a buffer, one
    assert min(sizes) >= 3 and any(full[b] and not full[b + 2] for a, e in zip(ends, ends[1:]) for b in range(a, e - 2))
    W = rand_pruned(rng, M, K, 0.004)
    for b in range(blocks):
        at = slice(128 * b, min(128 * b + 128, K))
        if full[b]:
            W[:, at] = rand_pruned(rng, M, at.stop - at.start, 0.9)
    L = cl.compress_layer(W, 6, 4, 128, 128, upload=True)
    planes = 2 * (blocks * 8 + 4) * cols * 16 * 2            # (four groups of sixteen columns are read ahead)
    assert cl.fc_workspace_bytes(L, B, cl.PATH_MFMA_BF16) == -(-planes // 256) * 256 + M * splits * cols * 4
    oW = oracle.dense_weights(oracle.compress_layer(W, 6, 4, 128, 128))
    X = rng.standard_normal((B, K)).astype(np.float32)
    Y = cl.compressed_fc_forward(L, torch.from_numpy(X).cuda(), None, relu=False, path=cl.PATH_MFMA_BF16).cpu().numpy()
    pick = np.unique(np.r_[0:B:31, B - 1])
    assert_close(Y[pick], fc_ref(oW, X[pick], None), False, product_rel=BF16X3)
    L.free()


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
