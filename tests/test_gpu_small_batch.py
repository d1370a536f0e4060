"""The small-batch kernel's one pass over a record, which starts where a table of the records'
positions says: position tables of 16 and of 32 bits a record (blocks of up to and of more than 65 536
cells), block widths that are a power of two and not, ragged last blocks, rows that span many
lanes' records and lanes that hold many rows, dense, sparse and empty layers; every batch tile, and layers
in one grid."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu

# rows, columns, block height and width, density, value and index bits
CASES = [(256, 1024, 256, 256, 0.07, 5, 4), (256, 1030, 256, 257, 0.07, 5, 4), (300, 2100, 256, 1000, 0.03, 5, 5), (130, 70000, 130, 70000, 0.002, 5, 8),
         (200, 333, 64, 48, 0.3, 8, 4), (130, 390, 128, 128, 1.0, 8, 5), (1, 500, 1, 128, 0.5, 5, 4), (257, 261, 128, 1, 0.2, 3, 3),
         (128, 256, 128, 128, 0.0, 5, 4)]


@pytest.mark.parametrize("M,K,bh,bw,d,r,k", CASES)
def test_one_pass(M, K, bh, bw, d, r, k):
    import torch
    rng = np.random.default_rng(M + K)
    W = rand_pruned(rng, M, K, d)
    L = cl.compress_layer(W, r, k, bh, bw, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, r, k, bh, bw))
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    for B in (1, 2, 3, 4, 8):
        X = rng.standard_normal((B, K)).astype(np.float32)
        Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
        Y = cl.compressed_fc_forward(L, Xd, bd, relu=False, path=cl.PATH_SPARSE)
        assert_close(Y.cpu().numpy(), fc_ref(oW, X, bias), False)
        assert torch.equal(Y, cl.compressed_fc_forward(L, Xd, bd, relu=False, path=cl.PATH_SPARSE))
    L.free()


def named_cells(L):
    """(row, column) of every entry of the layer, padding included, by its decoded indices."""
    M, K, bh, bw = (L.host_view()["desc"][n] for n in ("M", "K", "block_h", "block_w"))
    _, idx, bp, _ = (t.cpu().numpy().astype(np.int64) if t is not None else None for t in cl.decode_layer(L, want_dense=False))
    out = np.zeros((M, K), bool)
    per_row = -(-K // bw)
    for b in range(len(bp) - 1):
        r0, c0 = b // per_row * bh, b % per_row * bw
        pos = np.cumsum(idx[bp[b]:bp[b + 1]] + 1) - 1
        w = min(bw, K - c0)
        out[r0 + pos // w, c0 + pos % w] = True
    return out


# (the last two: one launch where four images and fewer allow)
@pytest.mark.parametrize("M,K,bh,bw,d,r,k", [(256, 1024, 256, 256, 0.07, 5, 4), (300, 2100, 256, 1000, 0.03, 5, 5), (200, 6000, 64, 48, 0.05, 8, 4),
                                             (300, 9000, 128, 128, 0.05, 5, 4), (256, 384, 128, 128, 0.05, 5, 4), (200, 333, 64, 48, 0.1, 8, 4)])
def test_values_that_are_not_finite_stay_in_their_rows(M, K, bh, bw, d, r, k):
    """A lane looks columns up past its own record's last entry: an output without an entry in a column has nothing of it."""
    import torch
    rng = np.random.default_rng(M + K)
    L = cl.compress_layer(rand_pruned(rng, M, K, d), r, k, bh, bw, upload=True)
    cells = named_cells(L)
    G = cl.LayerGroup([L])
    for B in (1, 2, 4, 8):
        X = rng.standard_normal((B, K)).astype(np.float32)
        bad = rng.choice(K, 4, replace=False)
        Z = X.copy()
        Z[B // 2, bad] = [np.inf, np.nan, -np.inf, np.inf]
        alone, grid = (lambda x: cl.compressed_fc_forward(L, x, path=cl.PATH_SPARSE)), (lambda x: G.forward(x[None])[0])
        for call in (alone, grid) if bh < 256 or B < 8 else (alone,):        # (a grid takes no more images than one tile has room for)
            want, got = (call(torch.from_numpy(a).cuda()).cpu().numpy() for a in (X, Z))
            touched = np.zeros((B, M), bool)
            touched[B // 2] = cells[:, bad].any(axis=1)
            assert touched.any() and not touched.all(axis=1).any()
            assert np.array_equal(got[~touched].view(np.uint32), want[~touched].view(np.uint32))
            assert not np.isfinite(got[touched]).any()
    L.free()


@pytest.mark.parametrize("B", [1, 2, 4, 8])
def test_one_pass_in_one_grid(B):
    import torch
    M, K, bh, bw = 300, 1100, 128, 100
    rng = np.random.default_rng(B)
    Ws = [rand_pruned(rng, M, K, d) for d in (0.1, 0.4, 0.01)]
    G = cl.LayerGroup([cl.compress_layer(W, 5, 4, bh, bw, upload=True) for W in Ws])
    X = rng.standard_normal((3, B, K)).astype(np.float32)
    Y = G.forward(torch.from_numpy(X).cuda()).cpu().numpy()
    for i, W in enumerate(Ws):
        assert_close(Y[i], fc_ref(oracle.dense_weights(oracle.compress_layer(W, 5, 4, bh, bw)), X[i], None), False)
