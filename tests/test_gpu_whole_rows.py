"""Small layers in one launch, a workgroup to a block row, where that is the faster form: block rows of no, one, sixteen, seventeen
and 48 chunks (the most) and of 49 (two launches), ragged last blocks, widths that are no power of two, positions
of 32 bits; to the last bit what the two launches give, which a group of layers in one grid takes."""
import numpy as np
import pytest

import oracle
import paper_1711_00244_amd as cl
from gates import assert_close, fc_ref
from test_host_library import rand_pruned

WAVES, ROUNDS = 16, 3                    # wavefronts of a workgroup, chunks that one of them takes at most

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
        plain = cl.compressed_fc_forward(L, Xd, None, relu=False, path=cl.PATH_SPARSE)
        assert torch.equal(plain, G.forward((Xd if B != 3 else torch.cat([Xd, Xd[:1]]))[None])[0, :B])


def chunks_of(L):
    """Chunks of the layer's largest block row."""
    return int(np.diff(np.asarray(L.host_view()["panel_chunk"]).astype(np.int64)).max())


def one_launch(L, Xd, forward):
    """Whether forward(workspace) ran the layer in one launch, which leaves no partial tiles in its workspace."""
    import torch
    ws = torch.full((max(256, cl.fc_workspace_bytes(L, Xd.shape[0], cl.PATH_SPARSE)),), 0xA5, dtype=torch.uint8, device="cuda")
    Y = forward(ws)
    torch.cuda.synchronize()
    return bool((ws == 0xA5).all()), Y


# blocks of `cols` columns and their density in a row of `blocks` of them: one launch for a call by itself, for a captured one
# (which has its launches made already: only GPU time counts there)
@pytest.mark.parametrize("M,bh,cols,blocks,d,B,plain,captured", [
    (1024, 128, 128, 8, 0.1, 1, True, False), (1024, 128, 128, 3, 0.1, 1, True, True), (512, 128, 128, 22, 0.018, 1, False, False),
    (96, 16, 16, 40, 0.5, 1, True, False), (96, 16, 16, 47, 0.5, 2, False, False), (96, 32, 100, 44, 0.1, 2, False, False), (96, 16, 16, 16, 0.5, 4, True, True),
    (96, 16, 16, 46, 0.5, 4, False, False), (32, 16, 16, 36, 0.5, 4, True, False), (32, 16, 16, 36, 0.5, 3, True, False), (16 * 128, 16, 16, 48, 0.5, 3, True, True)])
def test_one_launch_where_it_is_the_faster_one(M, bh, cols, blocks, d, B, plain, captured):
    import torch
    rng = np.random.default_rng(blocks)
    K = cols * blocks
    W = rand_pruned(rng, M, K, d)
    L = cl.compress_layer(W, 5, 4, bh, cols, upload=True)
    assert WAVES < chunks_of(L) <= WAVES * ROUNDS or plain and captured
    oW = oracle.dense_weights(oracle.compress_layer(W, 5, 4, bh, cols))
    X = rng.standard_normal((B, K)).astype(np.float32)
    Xd, out = torch.from_numpy(X).cuda(), torch.empty((B, M), device="cuda")
    two = cl.LayerGroup([L]).forward(Xd[None] if B != 3 else torch.cat([Xd, Xd[:1]])[None])[0, :B]

    def call(ws):
        return cl.compressed_fc_forward(L, Xd, None, relu=False, path=cl.PATH_SPARSE, out=out, workspace=ws)

    got, Y = one_launch(L, Xd, call)
    assert got == plain
    assert_close(Y.cpu().numpy(), fc_ref(oW, X), False)
    assert torch.equal(Y, two)
    g = torch.cuda.CUDAGraph()

    def replay(ws):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            call(ws)                                     # (what a first call loads is loaded)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        ws.fill_(0xA5)
        with torch.cuda.graph(g):
            call(ws)
        for _ in range(3):
            out.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, two)
        return out

    assert one_launch(L, Xd, replay)[0] == captured
    # behind another layer, and in front of one: the same values whatever the form
    for layers in ([L], [cl.compress_layer(np.eye(K, dtype=np.float32), 1, 8, 128, 128, codebook=np.array([0, 1], np.float32), upload=True), L]):
        if B > 1:                                        # (one image: the sum of the layer before is formed in another order)
            assert torch.equal(cl.compressed_fc_stack_forward(layers, Xd, relu_hidden=False, path=cl.PATH_SPARSE), two)


def test_one_launch_behind_full_image_tiles():
    """Nine to twelve images on small blocks: eight in two launches, the rest in one."""
    import torch
    rng = np.random.default_rng(9)
    M, K = 1000, 256
    W = rand_pruned(rng, M, K, 0.2)
    L = cl.compress_layer(W, 5, 4, 4, 16, upload=True)       # (so many that fc_rows_kernel does not take them)
    oW = oracle.dense_weights(oracle.compress_layer(W, 5, 4, 4, 16))
    bias = (rng.standard_normal(M) * 0.1).astype(np.float32)
    bd = torch.from_numpy(bias).cuda()
    for B in (9, 10, 11, 12):
        X = rng.standard_normal((B, K)).astype(np.float32)
        Xd = torch.from_numpy(X).cuda()
        Y = cl.compressed_fc_forward(L, Xd, bd, relu=True, path=cl.PATH_SPARSE)
        assert_close(Y.cpu().numpy(), fc_ref(oW, X, bias), True)
        one, rest = one_launch(L, Xd[8:], lambda ws: cl.compressed_fc_forward(L, Xd[8:], bd, relu=True, path=cl.PATH_SPARSE, workspace=ws))
        assert one and torch.equal(Y[8:], rest)
    L.free()


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
