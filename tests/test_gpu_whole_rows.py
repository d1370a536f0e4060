"""Small layers in one launch, a workgroup to a block row: block rows of no, one, sixteen, seventeen and 48 chunks (the most)
and of 49 (two launches), ragged last blocks, widths that are no power of two, positions of 32 bits; to the
last bit what the two launches give, which a group of layers in one grid still takes."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu

# rows, columns, block height and width, density, value and index bits
CASES = [(1024, 1024, 128, 128, 0.1, 5, 4), (300, 333, 128, 128, 0.3, 5, 4), (256, 256, 256, 256, 0.2, 5, 4), (257, 500, 128, 100, 0.05, 8, 5),
         (1, 64, 1, 64, 0.5, 5, 4), (100, 3000, 64, 3000, 0.02, 5, 8), (512, 2048, 128, 128, 0.002, 5, 4)] + [
             (100, 128 * n, 64, 128, 0.05, 5, 4) for n in (1, 16, 17, 32, 33, 48, 49)]


@pytest.mark.parametrize("M,K,bh,bw,d,r,k", CASES)
def test_whole_block_rows(M, K, bh, bw, d, r, k):
    import torch
    rng = np.random.default_rng(M + 3 * K)
    W = rand_pruned(rng, M, K, d)
    W[-(M % bh or bh):] = 0 if M > bh else W[-(M % bh or bh):]           # the last block row without a chunk
    L = cl.compress_layer(W, r, k, bh, bw, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, r, k, bh, bw))
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    G = cl.LayerGroup([L])
    for B in (1, 2, 3, 4):
        X = rng.standard_normal((B, K)).astype(np.float32)
        Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
        for relu in (False, True):
            Y = cl.compressed_fc_forward(L, Xd, bd, relu=relu, path=cl.PATH_SPARSE)
            assert_close(Y.cpu().numpy(), fc_ref(oW, X, bias), relu)
        if B != 3:
            plain = cl.compressed_fc_forward(L, Xd, None, relu=False, path=cl.PATH_SPARSE)
            assert torch.equal(plain, G.forward(Xd[None])[0])


@pytest.mark.parametrize("M,bh,n", [(2976, 1, 1), (2977, 1, 1), (3 * 3500, 3, 1), (4096, 1, 8), (4097, 1, 8), (4097, 1, 9)])
def test_many_block_rows(M, bh, n):
    """On both sides of the line between one launch and two, block rows of one, eight and nine chunks."""
    import torch
    rng = np.random.default_rng(M + n)
    K = 130 * n
    W = rand_pruned(rng, M, K, 0.05)
    W[::3, ::130] = 0.5                                       # (no block row without a chunk)
    L = cl.compress_layer(W, 5, 4, bh, 130, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, 5, 4, bh, 130))
    G = cl.LayerGroup([L])
    for B in (1, 2, 3):
        X = rng.standard_normal((B, K)).astype(np.float32)
        Xd = torch.from_numpy(X).cuda()
        Y = cl.compressed_fc_forward(L, Xd, None, relu=False, path=cl.PATH_SPARSE)
        assert_close(Y.cpu().numpy(), fc_ref(oW, X), False)
        if B != 3:
            assert torch.equal(Y, G.forward(Xd[None])[0])
    L.free()


def test_more_block_rows_than_a_launch_has_threads_for():
    """2^22 block rows: at 1024 threads each one more thread than a launch's 32 bits count, at the two launches'
    512 half of that."""
    import torch
    rng = np.random.default_rng(22)
    M, K = 1 << 22, 129
    rows = np.unique(np.concatenate([rng.integers(0, M, 999), [0, M - 1]]))
    W = np.zeros((M, K), np.float32)                         # (blocks above 128 columns: no tables for the other paths)
    W[rows] = rng.integers(-3, 4, (len(rows), K))
    L = cl.compress_layer(W, 3, 8, 1, K, codebook=np.array([0, 1, 2, 3, -1, -2, -3, 4], np.float32), upload=True)
    X = rng.integers(-8, 9, (1, K)).astype(np.float32)
    Y = cl.compressed_fc_forward(L, torch.from_numpy(X).cuda(), None, relu=False, path=cl.PATH_SPARSE).cpu().numpy()
    want = np.zeros((1, M), np.float32)
    want[:, rows] = X @ W[rows].T                            # (whole numbers below 2^24: exact in any order)
    assert np.array_equal(Y, want)
    L.free()
