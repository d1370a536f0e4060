"""The gathered convolution's split operands: sizes where its half blocks and row strips end,
values at the ends of the fp32 range, and what is not finite."""
import numpy as np
import pytest

import paper_1711_00244_amd as cl
from gates import assert_close, conv_ref

pytestmark = pytest.mark.gpu

IMAGES = 19                      # enough columns for the gathered form with a single block


def _layer(rng, geom, block_h, block_w, density=0.5):
    OC, K = geom["OC"], geom["C"] // geom["groups"] * geom["R"] * geom["S"]
    W = (rng.standard_normal((OC, K)) * (rng.random((OC, K)) < density)).astype(np.float32)
    L = cl.compress_layer(W, 8, 8, block_h, block_w, upload=True)
    return L, cl.decode_layer(L)[3].cpu().numpy()


def _geom(C, H, R, OC, groups=1):
    return dict(C=C, H=H, W=H, R=R, S=R, stride=1, pad=R // 2, groups=groups, OC=OC)


# input channels, filters, block height and width: one half block, both, a ragged last block with and
# without a second half, blocks of one half; strips of 32, 64, 96 and 128 rows, whole and not
@pytest.mark.parametrize("C,OC,bh,bw", [(7, 128, 128, 128), (8, 128, 128, 128), (15, 40, 64, 128), (20, 70, 96, 128), (22, 130, 128, 128),
                                        (29, 96, 96, 128), (9, 64, 64, 64), (16, 100, 128, 48), (64, 33, 64, 128)])
@pytest.mark.parametrize("path", ["f32", "bf16"])
def test_tile_edges(C, OC, bh, bw, path):
    import torch
    rng = np.random.default_rng(C * OC)
    geom = _geom(C, 30, 3, OC)
    L, W = _layer(rng, geom, bh, bw)
    X = rng.standard_normal((IMAGES, C, 30, 30)).astype(np.float32)
    Y = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False,
                                   path=cl.PATH_MFMA_BF16 if path == "bf16" else cl.PATH_MFMA_F32).cpu().numpy()
    # (two bf16 terms each: what is dropped is below 3 * 2^-16 of each product)
    assert_close(Y, conv_ref(W, X, geom), False, product_rel=3 * 2.0 ** -16 if path == "bf16" else 0.0)
    L.free()


def test_large_values_do_not_overflow():
    """Activations above the largest bf16 (3.39e38): the products stay in range with small weights."""
    import torch
    rng = np.random.default_rng(5)
    geom = _geom(8, 30, 3, 128)
    L, W = _layer(rng, geom, 128, 128)
    L.free()
    scale = np.float32(2.0 ** -30)
    L = cl.compress_layer(W * scale, 8, 8, 128, 128, upload=True)
    W = cl.decode_layer(L)[3].cpu().numpy()
    X = rng.standard_normal((IMAGES, 8, 30, 30)).astype(np.float32)
    X[:, :, 3::5, 2::7] = np.float32(3.4e38)
    X[:, :, 1::5, 2::7] = -np.float32(3.4e38)
    Y = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False).cpu().numpy()
    down = np.float32(2.0 ** -100)                                  # exact, and keeps the reference's sums in range
    assert np.isfinite(Y).all()
    assert_close(Y * down, conv_ref(W, X * down, geom), False)
    L.free()


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_not_finite(bad):
    """An infinity gives what fp32 arithmetic gives over the dense block: infinity of the product's
    sign with a weight, NaN with a zero; outputs that do not see it are as without it."""
    import torch
    rng = np.random.default_rng(6)
    geom = _geom(8, 30, 3, 128)
    L, W = _layer(rng, geom, 128, 128)
    X = rng.standard_normal((IMAGES, 8, 30, 30)).astype(np.float32)
    clean = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False).cpu().numpy()
    X[4, 5, 17, 11] = bad
    Y = cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False).cpu().numpy()
    taps = W.reshape(128, 8, 3, 3)[:, 5]
    seen = np.zeros(Y.shape, bool)
    for r in range(3):
        for s in range(3):
            y, x = 17 + 1 - r, 11 + 1 - s
            seen[4, :, y, x] = True
            with np.errstate(invalid="ignore"):
                want = np.float32(bad) * taps[:, r, s]
            assert np.array_equal(Y[4, :, y, x], want, equal_nan=True), (r, s)
    assert np.array_equal(Y[~seen], clean[~seen])
    L.free()
