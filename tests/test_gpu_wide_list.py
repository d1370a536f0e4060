"""The lists of the wide path, which a wavefront gathers in LDS before it writes them: chunks full to
the last place (every record of fifteen entries), halves of a block that hold all weights or none, one-column
second halves, widths that are no power of two, ragged last blocks, layers without a weight; the activations
laid out by the same launch, and by the layer before."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu


def _weights(rng, M, K, d, cols):
    W = rand_pruned(rng, M, K, d)
    if cols is not None:
        keep = np.zeros(K, bool)
        keep[np.arange(K) % 128 // 64 == cols] = True
        W = np.where(keep, W, 0).astype(np.float32)
    return W


# rows, columns, block height and width, density, half of a block's columns that holds weights, value and index bits
CASES = [(256, 512, 128, 128, 1.0, None, 4, 1), (130, 390, 128, 128, 0.3, None, 8, 5), (128, 256, 128, 128, 0.2, 0, 5, 4), (128, 256, 128, 128, 0.2, 1, 5, 4),
         (100, 195, 100, 65, 0.4, None, 5, 4), (257, 300, 64, 100, 1.0, None, 8, 8), (200, 333, 16, 48, 0.1, None, 5, 3), (1, 64, 1, 64, 0.5, None, 5, 4),
         (128, 256, 128, 128, 0.0, None, 5, 4)]


@pytest.mark.parametrize("M,K,bh,bw,d,cols,r,k", CASES)
def test_lists_of_the_wide_path(M, K, bh, bw, d, cols, r, k):
    import torch
    rng = np.random.default_rng(M + K + r)
    W = _weights(rng, M, K, d, cols)
    L = cl.compress_layer(W, r, k, bh, bw, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, r, k, bh, bw))
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    for B in (1, 70, 256):
        X = rng.standard_normal((B, K)).astype(np.float32)
        Y = cl.compressed_fc_forward(L, torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda(), relu=False, path=cl.PATH_SPARSE_WIDE)
        assert_close(Y.cpu().numpy(), fc_ref(oW, X, bias), False)
    L.free()


def test_lists_of_a_stack():
    import torch
    rng = np.random.default_rng(5)
    dims = [(256, 384, 1.0), (300, 256, 0.2), (128, 300, 0.0), (70, 128, 0.5), (64, 70, 1.0)]       # more layers than one launch decodes
    Ws = [rand_pruned(rng, m, k, d) for m, k, d in dims]
    layers = [cl.compress_layer(W, 5, 4, 128, 128, upload=True) for W in Ws]
    X = torch.from_numpy(rng.standard_normal((130, 384)).astype(np.float32)).cuda()
    Y = cl.compressed_fc_stack_forward(layers, X, path=cl.PATH_SPARSE_WIDE)
    a = X
    for i, L in enumerate(layers):
        a = cl.compressed_fc_forward(L, a, relu=i + 1 < len(layers), path=cl.PATH_SPARSE_WIDE)
    assert torch.equal(Y, a)
