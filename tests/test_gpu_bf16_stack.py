"""A stack on the bf16 path, where a layer's finishing kernel writes the next layer's split
activations, against its layers called one by one: the same sums in the same order, so the same bits."""
import numpy as np
import pytest

import paper_1711_00244_amd as cl

pytestmark = pytest.mark.gpu


# widths and block heights: plain rows (fused), a ragged last block and a block height that is no
# multiple of four (not fused), block rows of 96 with a ragged last one
@pytest.mark.parametrize("widths,heights", [((300, 384, 256, 70), (128, 128, 128)), ((256, 200, 128, 40), (128, 64, 128)),
                                            ((130, 256, 128, 33), (33, 100, 64)), ((129, 384, 512, 128), (96, 96, 4))])
@pytest.mark.parametrize("batch", [1, 31, 33, 130, 300])
def test_stack_is_its_layers(widths, heights, batch):
    import torch
    rng = np.random.default_rng(batch)
    layers, biases = [], []
    for K, M, bh in zip(widths, widths[1:], heights):
        W = (rng.standard_normal((M, K)) * (rng.random((M, K)) < 0.2)).astype(np.float32)
        layers.append(cl.compress_layer(W, 5, 4, bh, 128, upload=True))
        biases.append(torch.from_numpy(rng.standard_normal(M).astype(np.float32)).cuda())
    X = torch.from_numpy(rng.standard_normal((batch, widths[0])).astype(np.float32)).cuda()
    Y = cl.compressed_fc_stack_forward(layers, X, biases, path=cl.PATH_MFMA_BF16)
    want = X
    for i, (L, b) in enumerate(zip(layers, biases)):
        want = cl.compressed_fc_forward(L, want, b, relu=i + 1 < len(layers), path=cl.PATH_MFMA_BF16)
    assert torch.equal(Y, want)
    for L in layers:
        L.free()
