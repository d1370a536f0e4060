"""The convolution form whose operands are split beforehand (conv_prepare_kernel, conv_plane_kernel): where its
tiles, units of k and blocks end, which calls take it, and what is not finite."""
import numpy as np
import pytest

import paper_1711_00244_amd as cl
from gates import assert_close, conv_ref

pytestmark = pytest.mark.gpu


def _geom(C, H, R, OC, groups=1, stride=1, pad=None, S=None, W=None):
    return dict(C=C, H=H, W=W or H, R=R, S=S or R, stride=stride, pad=R // 2 if pad is None else pad, groups=groups, OC=OC)


def _layer(rng, geom, block_h, block_w, density=0.4, codebook=None):
    K = geom["C"] // geom["groups"] * geom["R"] * geom["S"]
    W = (rng.standard_normal((geom["OC"], K)) * (rng.random((geom["OC"], K)) < density)).astype(np.float32)
    L = cl.compress_layer(W, 8, 8, block_h, block_w, codebook=codebook, upload=True)
    return L, cl.decode_layer(L)[3].cpu().numpy()


def _terms_bytes(geom, batch, terms):
    """The least that a call of this form asks for: the activations' terms."""
    Cg = geom["C"] // geom["groups"]
    H, W = geom["H"] + 2 * geom["pad"], geom["W"] + 2 * geom["pad"]
    channels = 4 if Cg <= 4 else -(-Cg // 8) * 8
    return 2 * terms * batch * geom["groups"] * channels * H * (W + (W & 1 if Cg <= 4 else 0))


def _round256(n):
    return -(-n // 256) * 256


def _shapes(geom, batch, terms, workspace):
    """(rows of a tile, splits of the steps, images of a launch) for which a call of this form asks for `workspace` bytes.  (Tiles that cut
    a filter group into as many rows, whole tiles counted, cannot be told apart.)"""
    Cg, g, R, S = geom["C"] // geom["groups"], geom["groups"], geom["R"], geom["S"]
    P, Q = ((geom[n] + 2 * geom["pad"] - geom[f]) // geom["stride"] + 1 for n, f in (("H", "R"), ("W", "S")))
    steps = ((R * -(-S // 2) if Cg <= 4 else -(-Cg // 8) * R * S) + 1) // 2
    found = set()
    for rows in (128, 96, 64):
        tiles = g * -(-(geom["OC"] // g) // rows)
        left = workspace - _round256(tiles * rows * steps * terms * 32) - _round256(8 * steps)
        for imgs in {-(-batch // runs) for runs in range(1, batch + 1)}:
            part = left - _round256(_terms_bytes(geom, imgs, terms))
            if part == 0:
                found.add((rows, 1, imgs))
            for last in {imgs, batch % imgs or imgs}:                           # (the last launch can split more)
                one = tiles * rows * -(-last * P * Q // 128) * 128 * 4          # (a multiple of 256)
                if part > 0 and part % one == 0 and 2 <= part // one <= steps:
                    found.add((rows, part // one, imgs))
    return found


@pytest.mark.parametrize("geom,batch,path,takes", [
    # (us in this form and in the faster of the others)
    (_geom(3, 227, 11, 96, stride=4, pad=0), 64, "f32", True),              # 138, 170
    (_geom(384, 13, 3, 256, groups=2), 64, "f32", True),                    # 84, 90
    (_geom(102, 44, 11, 190, stride=4), 2, "f32", False),                   # 60, 47
    (_geom(379, 11, 11, 433, stride=4), 33, "f32", False),                  # 293, 245
    (_geom(508, 16, 11, 410), 2, "bf16", False),                            # 320, 201
    (_geom(32, 180, 5, 50, stride=4), 1, "bf16", False),                    # 31, 23
    (_geom(7, 95, 3, 42, stride=2), 13, "bf16", False)])                    # 16, 13
def test_which_calls_take_it(geom, batch, path, takes):
    L, _ = _layer(np.random.default_rng(1), geom, cl.conv_block_h(geom["OC"], geom["groups"], 128), 128)
    n = cl.conv_workspace_bytes(L, geom, batch, cl.PATH_MFMA_BF16 if path == "bf16" else cl.PATH_MFMA_F32)
    assert bool(_shapes(geom, batch, 2 if path == "bf16" else 3, n)) == takes
    L.free()


def _check(rng, geom, block, batch, path, density=0.4, imgs=None, tile=None):
    """tile: the rows of the call's tiles, its steps split among workgroups."""
    import torch
    L, W = _layer(rng, geom, *block, density=density)
    terms = 2 if path == "bf16" else 3
    p = cl.PATH_MFMA_BF16 if path == "bf16" else cl.PATH_MFMA_F32
    n = cl.conv_workspace_bytes(L, geom, batch, p)
    assert n >= _terms_bytes(geom, imgs or batch, terms)
    # (the other forms' scratch can be larger than the terms: what this form asks for, to the byte)
    shapes = {(rows, splits > 1) for rows, splits, launch in _shapes(geom, batch, terms, n) if launch == (imgs or batch)}
    assert shapes == {(tile, True)} if tile else shapes
    X = rng.standard_normal((batch, geom["C"], geom["H"], geom["W"])).astype(np.float32)
    bias = rng.standard_normal(geom["OC"]).astype(np.float32)
    Xd, bd = torch.from_numpy(X).cuda(), torch.from_numpy(bias).cuda()
    Y = cl.compressed_conv_forward(L, geom, Xd, bd, relu=True, path=p)
    again = cl.compressed_conv_forward(L, geom, Xd, bd, relu=True, path=p)
    assert torch.equal(Y, again)
    Y = Y.cpu().numpy()
    # filters of the first and last rows of tiles and groups, the first and last image and one between
    OC, g, Cg = geom["OC"], geom["groups"], geom["C"] // geom["groups"]
    per = OC // g
    some = sorted({0, batch // 2, batch - 1})
    for grp in range(g):
        rows = sorted({r for r in (0, 31, 63, 64, 95, 96, 127, 128, per - 1) if r < per})
        sub = dict(geom, C=Cg, OC=len(rows), groups=1)
        at = np.array(rows) + grp * per
        ref = conv_ref(np.ascontiguousarray(W[at]), np.ascontiguousarray(X[some][:, grp * Cg:(grp + 1) * Cg]), sub, bias[at])
        # (two bf16 terms each: what is dropped is below 3 * 2^-16 of each product)
        assert_close(Y[some][:, at], ref, True, product_rel=3 * 2.0 ** -16 if path == "bf16" else 0.0)
    L.free()


CASES = [
    # tiles of 128, 96 and 64 filters, whole and not; channels that fill their last group of eight, and not
    (_geom(40, 56, 3, 128), (128, 128), 16), (_geom(41, 56, 3, 130), (128, 128), 16), (_geom(33, 56, 3, 96), (96, 128), 20),
    (_geom(63, 57, 3, 64), (64, 128), 24), (_geom(65, 40, 3, 200), (128, 128), 24),
    # an odd number of units (25 taps of one group of eight, 9 of three), taps by rows and columns
    (_geom(8, 64, 5, 130), (128, 128), 24), (_geom(24, 56, 3, 250), (128, 128), 16),
    (_geom(24, 48, 1, 190, S=7, pad=3), (128, 128), 24),
    # four channels to a pixel: odd and even numbers of taps, odd and even widths, two filter groups
    (_geom(3, 129, 11, 96, stride=2, pad=0), (96, 128), 48), (_geom(4, 65, 3, 250), (128, 128), 64), (_geom(3, 80, 4, 250, pad=1), (128, 128), 40),
    (_geom(8, 61, 5, 256, groups=2), (128, 128), 32),
    # filter groups with filters of their own tiles; strides; blocks of other widths and heights
    (_geom(96, 27, 5, 256, groups=2), (128, 128), 16), (_geom(384, 13, 3, 384, groups=2), (96, 128), 48), (_geom(48, 90, 3, 160, stride=2), (128, 128), 24),
    (_geom(40, 56, 3, 128), (64, 48), 20), (_geom(40, 56, 3, 120), (24, 128), 20), (_geom(20, 40, 11, 96), (96, 128), 16),
]


@pytest.mark.parametrize("geom,block,batch", CASES)
@pytest.mark.parametrize("path", ["f32", "bf16"])
def test_edges(geom, block, batch, path):
    _check(np.random.default_rng(geom["C"] * geom["OC"] + batch), geom, block, batch, path)


@pytest.mark.parametrize("geom,block,batch,tile", [
    (_geom(520, 14, 3, 440), (128, 128), 20, 128), (_geom(505, 15, 11, 70), (72, 128), 8, 96), (_geom(1000, 12, 3, 540, groups=2), (90, 128), 24, 96),
    (_geom(470, 14, 3, 270), (128, 128), 16, 64)])
@pytest.mark.parametrize("path", ["f32", "bf16"])
def test_steps_split_among_workgroups(geom, block, batch, tile, path):
    """Few columns and many units: each tile with its partial tiles added up, also of two filter groups."""
    _check(np.random.default_rng(tile), geom, block, batch, path, tile=tile)


@pytest.mark.parametrize("geom,block,batch,imgs", [
    # terms of all images 300 MB; one image's terms 290 MB; images of 2^18 pixels, at most eight to a launch; a last launch of fewer images
    (_geom(64, 112, 3, 128), (128, 128), 60, 30), (_geom(480, 316, 1, 64, pad=0), (64, 128), 2, 1), (_geom(4, 512, 3, 96), (96, 128), 10, 5),
    # (twice; then also in three splits of the steps where the first launch has two)
    (_geom(72, 200, 3, 64), (64, 128), 25, 13), (_geom(520, 80, 3, 64), (64, 128), 17, 9)])
def test_images_in_groups(geom, block, batch, imgs):
    """Scratch that grows with the images stays below 256 MB, or one image's; the images are taken in groups, the weights split with the
    first."""
    rng = np.random.default_rng(imgs)
    L, _ = _layer(rng, geom, *block)
    assert {s[2] for s in _shapes(geom, batch, 3, cl.conv_workspace_bytes(L, geom, batch))} == {imgs}
    assert _terms_bytes(geom, imgs, 3) <= 256 << 20 or imgs == 1
    L.free()
    _check(rng, geom, block, batch, "f32", imgs=imgs)


@pytest.mark.parametrize("density", [0.0, 0.02, 1.0])
def test_densities(density):
    """Blocks without a chunk, of one, and of many (the chunks that a workgroup takes are counted from their carries)."""
    _check(np.random.default_rng(7), _geom(41, 56, 3, 130), (128, 128), 16, "f32", density)


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("geom,batch", [(_geom(41, 56, 3, 130), 16), (_geom(3, 80, 5, 250), 40)])
def test_not_finite(geom, batch, bad):
    """What is not finite gives what fp32 gives over the dense block (a tap shared between two units once, not twice),
    and outputs that do not see it are as without it (slots and units that are not there are zeros on both sides)."""
    import torch
    rng = np.random.default_rng(6)
    L, W = _layer(rng, geom, 128, 128)
    R, pad, OC = geom["R"], geom["pad"], geom["OC"]
    X = rng.standard_normal((batch, geom["C"], geom["H"], geom["W"])).astype(np.float32)
    assert _shapes(geom, batch, 3, cl.conv_workspace_bytes(L, geom, batch))
    clean = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False).cpu().numpy()
    X[4, geom["C"] - 1, 17, 11] = bad
    Y = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False).cpu().numpy()
    taps = W.reshape(OC, geom["C"], R, R)[:, -1]
    seen = np.zeros(Y.shape, bool)
    for r in range(R):
        for s in range(R):
            y, x = 17 + pad - r, 11 + pad - s
            seen[4, :, y, x] = True
            with np.errstate(invalid="ignore"):
                want = np.float32(bad) * taps[:, r, s]
            assert np.array_equal(Y[4, :, y, x], want, equal_nan=True), (r, s)
    assert np.array_equal(Y[~seen], clean[~seen])
    L.free()


def test_codebooks_that_do_not_split():
    """Half a weight of 2^-110 is below what three terms hold: where two units share a tap such a layer goes the other way."""
    import torch
    rng = np.random.default_rng(8)
    cb = np.concatenate([[0.0], np.linspace(1, 2, 255) * 2.0 ** -110 * (1 + 2.0 ** -20)]).astype(np.float32)
    geom, batch = _geom(3, 80, 5, 250), 40
    L, W = _layer(rng, geom, 128, 128, codebook=cb)
    n = cl.conv_workspace_bytes(L, geom, batch)
    assert n < _terms_bytes(geom, batch, 3) and not _shapes(geom, batch, 3, n)
    X = (rng.standard_normal((batch, 3, 80, 80)) * 2.0 ** 100).astype(np.float32)
    Y = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda()).cpu().numpy()
    up = np.float32(2.0 ** 20)
    rows, imgs = np.array([0, 249]), [0, batch - 1]
    assert_close(Y[imgs][:, rows] * up, conv_ref(np.ascontiguousarray(W[rows]) * up, np.ascontiguousarray(X[imgs]), dict(geom, OC=2)), False)
    L.free()


def test_scratch_of_the_other_forms():
    """With less scratch than this form takes the call runs in the gathered form, and with less than that in the compact one;
    below the least it is refused."""
    import torch
    rng = np.random.default_rng(9)
    geom, batch = _geom(96, 27, 5, 256, groups=2), 16
    L, W = _layer(rng, geom, 128, 128)
    X = torch.from_numpy(rng.standard_normal((batch, 96, 27, 27)).astype(np.float32)).cuda()
    full, least = cl.conv_workspace_bytes(L, geom, batch), cl.conv_workspace_bytes(L, geom, batch, compact=True)
    assert least < full and _shapes(geom, batch, 3, full)
    rows, imgs = np.array([0, 127]), [0, batch - 1]
    ref = conv_ref(np.ascontiguousarray(W[rows]), np.ascontiguousarray(X.cpu().numpy()[imgs][:, :48]), dict(geom, C=48, OC=2, groups=1))
    for n in (full, full - 256, least):
        Y = cl.compressed_conv_forward(L, geom, X, workspace=torch.empty(n, dtype=torch.uint8, device="cuda")).cpu().numpy()
        assert_close(Y[imgs][:, rows], ref, False)
    with pytest.raises(cl.CLError):
        cl.compressed_conv_forward(L, geom, X, workspace=torch.empty(least - 256, dtype=torch.uint8, device="cuda"))
    L.free()


def test_scratch_without_split_operands():
    """The gathered form can be asked for by its scratch - decoded blocks, the row table, partial tiles - and is what then runs; a call
    that splits nothing asks for the same either way."""
    import torch
    from paper_1711_00244_amd import network
    rng = np.random.default_rng(10)
    geom, batch = _geom(96, 27, 5, 256, groups=2), 16
    L, W = _layer(rng, geom, 128, 128)
    full, n = cl.conv_workspace_bytes(L, geom, batch), cl.conv_workspace_bytes(L, geom, batch, unsplit=True)
    blocks, columns = 2 * 10, -(-batch * 27 * 27 // 128) * 128
    part = n - blocks * 128 * 128 * 4 - 10 * 128 * 8
    assert n != full and part % (256 * columns * 4) == 0 and part // (256 * columns * 4) in range(11)
    assert cl.conv_workspace_bytes(L, geom, 1) == cl.conv_workspace_bytes(L, geom, 1, unsplit=True)
    X = torch.from_numpy(rng.standard_normal((batch, 96, 27, 27)).astype(np.float32)).cuda()
    fast = network.ConvOp("conv", L, geom, (128, 128))
    op = network.unsplit_copy(network.NetworkRunner([fast], (96, 27, 27))).layers[0]
    assert op.ws_bytes(batch, None) == n
    Y = op.forward(X)
    assert torch.equal(Y, cl.compressed_conv_forward(L, geom, X, relu=True, workspace=torch.empty(n, dtype=torch.uint8, device="cuda")))
    assert not torch.equal(Y, fast.forward(X))               # (the sums run in another order)
    rows, imgs = np.array([0, 127]), [0, batch - 1]
    sub = dict(geom, C=48, OC=2, groups=1)
    assert_close(Y.cpu().numpy()[imgs][:, rows], conv_ref(np.ascontiguousarray(W[rows]), np.ascontiguousarray(X.cpu().numpy()[imgs][:, :48]), sub), True)
    L.free()
