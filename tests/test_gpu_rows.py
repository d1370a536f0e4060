"""The sparse path's kernel for more than a few images (fc_rows_kernel) against the oracle, under
both gates: batches on both sides of its image tiles and of the hand-over from the small-batch
kernel, ragged last blocks in both directions (K no multiple of four), narrow and low blocks,
rows and blocks without entries, rows with more entries than a quarter wavefront takes at a time,
blocks of more chunks than a workgroup has wavefronts, and an index table larger than the value table; results the
same every run, and independent of a non-finite activation in a column that no surviving weight of
the row names."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

pytestmark = pytest.mark.gpu

CASES = [(300, 521, 128, 128, 0.09, 5, 4), (515, 700, 128, 128, 0.001, 5, 4), (256, 1024, 128, 128, 0.25, 5, 4), (130, 390, 128, 128, 1.0, 8, 5),
         (200, 333, 64, 48, 0.2, 5, 4), (257, 261, 128, 20, 0.1, 5, 5), (140, 2050, 100, 128, 0.04, 3, 8), (128, 128, 128, 128, 0.0, 5, 4)]


@pytest.mark.parametrize("M,K,bh,bw,d,r,k", CASES)
@pytest.mark.parametrize("B", [9, 16, 17, 32, 33, 64, 65, 130])
def test_rows_kernel(M, K, bh, bw, d, r, k, B):
    import torch
    rng = np.random.default_rng(M + K + B)
    W = rand_pruned(rng, M, K, d)
    L = cl.compress_layer(W, r, k, bh, bw, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, r, k, bh, bw))
    X = np.maximum(rng.standard_normal((B, K)), 0).astype(np.float32)
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
    for b, relu in ((None, False), (bd, True)):
        Y = cl.compressed_fc_forward(L, Xd, b, relu=relu, path=cl.PATH_SPARSE)
        assert_close(Y.cpu().numpy(), fc_ref(oW, X, None if b is None else bias), relu)
        assert torch.equal(Y, cl.compressed_fc_forward(L, Xd, b, relu=relu, path=cl.PATH_SPARSE))
    L.free()


def test_rows_kernel_keeps_infinities_to_their_rows():
    import torch
    rng = np.random.default_rng(3)
    W = rand_pruned(rng, 200, 300, 0.02)
    W[:, 77] = 0.0
    W[9, :] = 0.0
    L = cl.compress_layer(W, 5, 4, 128, 128, upload=True)
    X = rng.random((12, 300)).astype(np.float32)
    want = cl.compressed_fc_forward(L, torch.from_numpy(X).cuda(), path=cl.PATH_SPARSE)
    X[3, 77] = np.inf
    got = cl.compressed_fc_forward(L, torch.from_numpy(X).cuda(), path=cl.PATH_SPARSE)
    val, idx, bp, dense = cl.decode_layer(L)
    # padding entries may name column 77; the kernel drops them
    assert torch.equal(got, want) and not bool(dense[:, 77].any())


# blocks of fewer than 64 x 64 cells, more than 12 of them to a CU of 256: the small-batch kernel up to 16
# images; fewer blocks, larger ones or more images: this one
@pytest.mark.parametrize("M,K,bh,bw,small", [(1040, 8192, 16, 128, True), (1040, 8192, 32, 64, True), (530, 8192, 32, 32, True), (1000, 4096, 16, 128, False),
                                             (1040, 8192, 64, 64, False)])
def test_kernel_by_block_size(M, K, bh, bw, small):
    """Which kernel it is shows in the scratch: the small-batch kernel's is the same for 8 and 16 images."""
    import torch
    rng = np.random.default_rng(bh + bw)
    W = rand_pruned(rng, M, K, 0.09)
    L = cl.compress_layer(W, 5, 4, bh, bw, upload=True)
    oW = oracle.dense_weights(oracle.compress_layer(W, 5, 4, bh, bw))
    need = {B: cl.fc_workspace_bytes(L, B, cl.PATH_SPARSE) for B in (8, 9, 16, 17)}
    assert (need[9] == need[8] and need[16] == need[8]) == small and need[17] != need[8], need
    for B in (9, 16, 17):
        X = np.maximum(rng.standard_normal((B, K)), 0).astype(np.float32)
        Xd = torch.from_numpy(X).cuda()
        ref = fc_ref(oW, X)
        for path in (cl.PATH_SPARSE, cl.PATH_AUTO):
            assert_close(cl.compressed_fc_forward(L, Xd, path=path).cpu().numpy(), ref, False)
    L.free()


def _device_bytes(L):
    import torch
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    L.upload()
    return before - torch.cuda.mem_get_info()[0]


@pytest.mark.parametrize("block", [(128, 128), (32, 128), (16, 16), (8, 8)])
def test_tables_in_proportion(block):
    """What a layer takes on the device beside its stored form: per block the 34 list positions of the
    large-batch path, its first entry and first chunk, and the lookup tables, which are left out
    above half the records' size (and a mebibyte); per chunk two list positions."""
    import torch
    W = rand_pruned(np.random.default_rng(4), 4096, 4096, 0.09)
    L = cl.compress_layer(W, 5, 4, *block)
    st = L.stats()
    tables = st["n_blocks"] * (34 * 4 + 4) + st["n_chunks"] * 8 + 2 * max(st["payload_bytes"] // 2, 1 << 20) + st["lut_bytes"]
    assert _device_bytes(L) <= st["model_bytes"] + tables + (2 << 20)          # (allocations come in pieces of 2 MiB)
    L.free()


def _one_full_block():
    """A layer whose blocks hold next to nothing, but for one that is full."""
    rng = np.random.default_rng(11)
    W = np.zeros((33 * 128, 100 * 128), np.float32)
    W[rng.integers(0, W.shape[0], 20000), rng.integers(0, W.shape[1], 20000)] = 0.02
    W[:128, 256:384] = rng.standard_normal((128, 128)) * 0.02
    return W


@pytest.mark.parametrize("make,block", [(lambda: rand_pruned(np.random.default_rng(5), 1040, 4096, 0.09), (8, 8)), (_one_full_block, (128, 128))],
                         ids=["small blocks", "one full block"])
def test_layers_without_the_lookup_tables(make, block):
    """They run on the small-batch kernel (its scratch is the same for any batch from 8 on), decode chunk
    by chunk, and give what the oracle gives."""
    import torch
    W = make()
    L = cl.compress_layer(W, 5, 4, *block, upload=True)
    m = oracle.compress_layer(W, 5, 4, *block)
    oW = oracle.dense_weights(m)
    assert len({cl.fc_workspace_bytes(L, B, cl.PATH_SPARSE) for B in (8, 9, 64)}) == 1
    val, idx, bp, dense = cl.decode_layer(L)
    oval, oidx, obp = oracle.decode_layer(m)
    assert np.array_equal(val.cpu().numpy(), oval) and np.array_equal(idx.cpu().numpy(), oidx) and np.array_equal(bp.cpu().numpy(), obp)
    assert np.array_equal(dense.cpu().numpy(), oW)
    rng = np.random.default_rng(6)
    X = np.maximum(rng.standard_normal((20, W.shape[1])), 0).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    ref = fc_ref(oW, X)
    for path in (cl.PATH_SPARSE, cl.PATH_AUTO):
        assert_close(cl.compressed_fc_forward(L, Xd, path=path).cpu().numpy(), ref, False)
    L.free()


# M, K: a batch in runs of four images a lane (1024 images of 4096 rows fill the scratch); of two and of
# one (so many rows that 63 and 31 images do); and one that leaves the path to the small-batch kernel
@pytest.mark.parametrize("M,K,B", [(4096, 260, 1023), (4096, 260, 1025), (4096, 260, 2100), (66000, 24, 200), (130000, 24, 70), (270000, 12, 20)])
def test_scratch_is_bounded(M, K, B):
    """The path's scratch does not grow with the batch, so the entry point without a workspace takes
    any; the images of every run come out as the oracle has them, and as a call with a workspace has."""
    import torch
    rng = np.random.default_rng(B)
    W = rand_pruned(rng, M, K, 0.1)
    L = cl.compress_layer(W, 5, 4, 128, 128, upload=True)
    assert cl.fc_workspace_bytes(L, B, cl.PATH_SPARSE) <= cl.STATIC_SCRATCH_BYTES
    oW = oracle.dense_weights(oracle.compress_layer(W, 5, 4, 128, 128))
    X = np.maximum(rng.standard_normal((B, K)), 0).astype(np.float32)
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
    out = torch.full((B, M), -7.0, device="cuda")
    cl.compressed_fc_forward_static(L, Xd, out, bd, relu=True, path=cl.PATH_SPARSE)
    assert torch.equal(out, cl.compressed_fc_forward(L, Xd, bd, relu=True, path=cl.PATH_SPARSE))
    rows = np.concatenate([np.arange(min(M, 300)), np.arange(max(0, M - 300), M)])
    assert_close(out.cpu().numpy()[:, rows], fc_ref(oW[rows], X, bias[rows]), True)
    # (the library's own choice of path: what it does not refuse with a workspace of that size runs here too)
    if cl.fc_workspace_bytes(L, B) <= cl.STATIC_SCRATCH_BYTES:
        cl.compressed_fc_forward_static(L, Xd, out, bd, relu=True)
        assert_close(out.cpu().numpy()[:, rows], fc_ref(oW[rows], X, bias[rows]), True)
    L.free()


def test_a_stack_chooses_its_paths_together():
    """Where the first layer of a stack is on the wide path, the second hands and is handed its
    activations and shares the decoding launch there: it stays on that path, which alone it would
    leave for this kernel.  Bit for bit the chain of the paths named; all layers on this kernel at 64."""
    import torch
    from paper_1711_00244_amd import workloads as wl
    layers = []
    for li in range(3):
        spec, W = wl.layer_weights(3, li)
        layers.append(cl.compress_layer(W, spec.r, spec.k, 128, 128, upload=True))
    for B, paths in ((64, [cl.PATH_SPARSE] * 3), (96, [cl.PATH_SPARSE_WIDE, cl.PATH_SPARSE_WIDE, cl.PATH_MFMA_F32]),
                     (128, [cl.PATH_SPARSE_WIDE, cl.PATH_SPARSE_WIDE, cl.PATH_MFMA_F32])):
        a = torch.from_numpy(wl.activations(3, B)).cuda()
        Y = cl.compressed_fc_stack_forward(layers, a)
        for li in range(3):
            a = cl.compressed_fc_forward(layers[li], a, relu=li < 2, path=paths[li])
        assert torch.equal(Y, a), B
    for L in layers:
        L.free()


# where CL_PATH_AUTO goes to this kernel and where it leaves it: a dense and a sparse layer, images on both sides of the line
@pytest.mark.parametrize("M,K,d,paths", [(1000, 4096, 0.25, {16: cl.PATH_SPARSE, 65: cl.PATH_SPARSE, 128: cl.PATH_SPARSE, 256: cl.PATH_MFMA_F32}),
                                         (4096, 4096, 0.09, {16: cl.PATH_SPARSE, 128: cl.PATH_SPARSE, 256: cl.PATH_SPARSE_WIDE}),
                                         (4096, 4096, 0.3, {16: cl.PATH_SPARSE, 128: cl.PATH_MFMA_F32}), (384, 500, 0.1, {64: cl.PATH_MFMA_F32})])
def test_auto_path(M, K, d, paths):
    import torch
    rng = np.random.default_rng(K)
    L = cl.compress_layer(rand_pruned(rng, M, K, d), 5, 4, 128, 128, upload=True)
    for B, path in paths.items():
        assert cl.fc_resolved_path(L, B) == path, B
        assert cl.fc_workspace_bytes(L, B) == cl.fc_workspace_bytes(L, B, path)
        X = torch.from_numpy(rng.standard_normal((B, K)).astype(np.float32)).cuda()
        assert torch.equal(cl.compressed_fc_forward(L, X), cl.compressed_fc_forward(L, X, path=path))
    L.free()
