"""cl_decode_layer's one-launch kernel for blocks of at most 128 x 128 against the oracle: sizes on
and off four columns, narrow, low and ragged blocks, blocks of no chunk and of more chunks than a
workgroup has wavefronts, outputs that begin on any byte, and each output left out."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu

CASES = [(300, 521, 128, 128, 0.09, 5, 4), (515, 700, 128, 128, 0.001, 5, 4), (256, 384, 128, 128, 1.0, 8, 5), (200, 333, 64, 48, 0.2, 5, 4),
         (257, 260, 128, 20, 0.1, 5, 5), (140, 1028, 100, 126, 0.04, 3, 8), (128, 128, 128, 128, 0.0, 5, 4), (37, 45, 5, 3, 0.3, 3, 2)]


@pytest.mark.parametrize("M,K,bh,bw,d,r,k", CASES)
def test_decode_blocks(M, K, bh, bw, d, r, k):
    import torch
    from paper_1711_00244_amd.binding import _check, _stream, lib
    rng = np.random.default_rng(M * K)
    W = rand_pruned(rng, M, K, d)
    L = cl.compress_layer(W, r, k, bh, bw, upload=True)
    o = oracle.compress_layer(W, r, k, bh, bw)
    val, idx, bp, dense = cl.decode_layer(L)
    np.testing.assert_array_equal(dense.cpu().numpy(), oracle.dense_weights(o))
    want = [t.cpu().numpy() for t in (val, idx, bp)] + [dense.cpu().numpy()]
    for got, sym in zip(want, oracle.decode_layer(o)):
        np.testing.assert_array_equal(got, sym)
    n, nb = val.numel(), bp.numel()
    for off in (1, 7, 8, 13):                       # each output by itself, at another place, nothing written round it
        for which in range(4):
            buf = torch.full(((n, n, 4 * nb, 4 * M * K)[which] + 64,), 0xA5, dtype=torch.uint8, device="cuda")
            at = off if which < 2 else 4 * off
            ptrs = [None] * 4
            ptrs[which] = buf.data_ptr() + at
            _check(lib().cl_decode_layer(L.handle, *ptrs, _stream()))
            got = buf.cpu().numpy()
            size = want[which].nbytes
            assert (got[:at] == 0xA5).all() and (got[at + size:] == 0xA5).all()
            np.testing.assert_array_equal(got[at:at + size], want[which].reshape(-1).view(np.uint8))
    L.free()


def test_large_dense_matrix():
    """A dense matrix of more than 64 MiB, ragged blocks on both edges."""
    rng = np.random.default_rng(64)
    W = rand_pruned(rng, 4133, 4148, 0.01)
    L = cl.compress_layer(W, 5, 4, 128, 128, upload=True)
    dense = cl.decode_layer(L)[3].cpu().numpy()
    assert dense.nbytes > 64 << 20
    np.testing.assert_array_equal(dense, oracle.dense_weights(oracle.compress_layer(W, 5, 4, 128, 128)))
    L.free()
