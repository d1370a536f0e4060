"""The host side's work shared among threads: layers large enough for several of them (and
one just below) come out as the oracle's entries, whatever the shape gives the threads to
share - one block row, one block column, ragged blocks, duplicate codebook values -
and the checksum computed in pieces is the plain FNV-1a of the stored bytes."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from test_host_library import cross_decode, rand_pruned

SHAPES = [(1, 700001, 1, 128, 0.1, 5, 4), (600011, 1, 128, 1, 0.1, 5, 4), (777, 1001, 128, 128, 0.09, 5, 4), (700, 900, 96, 100, 0.4, 8, 5),
          (4096, 300, 4096, 1, 0.05, 5, 2), (511, 1025, 128, 128, 0.0, 5, 4)]


@pytest.mark.parametrize("own_codebook", [False, True])
@pytest.mark.parametrize("M,K,bh,bw,d,r,k", SHAPES)
def test_threads_give_the_oracles_entries(M, K, bh, bw, d, r, k, own_codebook):
    rng = np.random.default_rng(M + K)
    W = rand_pruned(rng, M, K, d)
    cb = None
    if own_codebook:
        cb = np.concatenate([[0], rng.standard_normal((1 << r) - 1) * 0.02]).astype(np.float32)
        cb[7] = cb[3]                            # equal values: the lower index wins
    L = cl.compress_layer(W, r, k, bh, bw, codebook=cb)
    m = oracle.compress_layer(W, r, k, bh, bw, codebook=cb, keep=True)
    val, idx, bp = cross_decode(L)
    assert np.array_equal(val, m.extra["val"]) and np.array_equal(idx, m.extra["idx"]) and np.array_equal(bp, m.extra["block_ptr"])
    L2 = cl.layer_deserialize(L.serialize())
    a, b = L.host_view(), L2.host_view()
    assert L.stats() == L2.stats() and all(np.array_equal(a[x], b[x]) for x in ("chunk_nz", "chunk_half", "group_ptr", "records") if a[x] is not None)


@pytest.mark.parametrize("M,K,d", [(300, 512, 0.5), (512, 1024, 0.5), (1001, 777, 0.31)])
def test_checksum_in_pieces_is_plain_fnv1a(M, K, d):
    img = cl.compress_layer(rand_pruned(np.random.default_rng(5), M, K, d), 5, 4, 128, 128).serialize()
    hdr = int.from_bytes(img[12:16], "little")
    h = 1469598103934665603
    for byte in img[hdr:]:
        h = ((h ^ byte) * 1099511628211) & (2 ** 64 - 1)
    assert img[hdr - 8:hdr] == h.to_bytes(8, "little")
    bad = bytearray(img)
    bad[-3] ^= 4
    with pytest.raises(cl.CLError):
        cl.layer_deserialize(bytes(bad))


def test_a_non_finite_weight_is_named_whichever_thread_meets_it():
    W = rand_pruned(np.random.default_rng(6), 900, 1000, 0.1)
    W[613, 7] = np.nan
    W[40, 999] = -np.inf
    with pytest.raises(cl.CLError, match="element 40999"):
        cl.compress_layer(W, 5, 4, 128, 128)
