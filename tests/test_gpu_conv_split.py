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


def _one_by_one(rng, n, codebook=None, sigma=1.0):
    """A 1 x 1 convolution whose outputs are sums of n products, and its dense weights."""
    geom = _geom(n, 30, 1, 64)
    W = (rng.standard_normal((64, n)) * sigma).astype(np.float32)
    L = cl.compress_layer(W, 8, 8, 128, 128, codebook=codebook, upload=True)
    return geom, L, cl.decode_layer(L)[3].cpu().numpy().astype(np.float64)


def _run(L, geom, X):
    import torch
    return cl.compressed_conv_forward(L, geom, torch.from_numpy(X).cuda(), relu=False).cpu().numpy().astype(np.float64)


def _sums(W, X):
    return np.einsum("oc,nchw->nohw", W, X.astype(np.float64))


@pytest.mark.parametrize("n", [1, 2, 3])
@pytest.mark.parametrize("spread", ["normal", "near a power of two"])
def test_short_sums(n, spread):
    """One to three products: no more than the rounding of that many fp32 multiply-adds, n * 2^-24 of
    the sum of magnitudes.  (The seven products beside x1 w1 add up to less than 2^-6 of it, and each of
    their additions rounds by up to 2^-23 of that, in whatever manner the matrix cores round: with
    what is left out, less than 14 * 2^-30 + 2^-32 < 2^-2 * 2^-24.)"""
    rng = np.random.default_rng(n)
    if spread == "normal":
        geom, L, W = _one_by_one(rng, n)
        X = rng.standard_normal((IMAGES, n, 30, 30)).astype(np.float32)
    else:       # where a relative error weighs most: mantissas just above 1
        near = lambda shape: ((1 + rng.random(shape) * 2.0 ** -5) * 2.0 ** rng.integers(-3, 3, shape)).astype(np.float32)
        cb = np.concatenate([[0], np.sort(near(255))]).astype(np.float32)
        geom, L, W = _one_by_one(rng, n, cb)
        X = near((IMAGES, n, 30, 30))
    err = np.abs(_run(L, geom, X) - _sums(W, X))
    assert float((err / _sums(np.abs(W), np.abs(X))).max()) <= (n + 0.25) * 2.0 ** -24
    L.free()


@pytest.mark.parametrize("e", [90, 109, 114, 122, 130])
def test_small_activations(e):
    """Values around 2^-e: those of 2^-110 and more exact, smaller ones to the nearest multiple of
    bf16's smallest number, 2^-133.  (Weights around 2^30, so that the results are normal numbers.)"""
    rng = np.random.default_rng(e)
    n = 3
    geom, L, W = _one_by_one(rng, n, sigma=2.0 ** 30)
    X = (rng.standard_normal((IMAGES, n, 30, 30)) * 2.0 ** -e).astype(np.float32)
    err = np.abs(_run(L, geom, X) - _sums(W, X))
    lost = np.where(np.abs(X) < 2.0 ** -110, 2.0 ** -134, 0.0)
    assert (err <= (n + 0.25) * 2.0 ** -24 * _sums(np.abs(W), np.abs(X)) + _sums(np.abs(W), lost)).all()
    L.free()


@pytest.mark.parametrize("low", [2.0 ** -112, 2.0 ** -120, -0.0])
def test_codebooks_that_do_not_split(low):
    """Weights below 2^-110, and a codebook's -0, go the other way: exact to fp32's rounding."""
    rng = np.random.default_rng(8)
    cb = np.concatenate([[low if low == 0 else 0.0], np.linspace(-1, 1, 255) * (low if low else 1.0) * (1 + 2.0 ** -20)]).astype(np.float32)
    geom, L, W = _one_by_one(rng, 3, cb, sigma=low if low else 1.0)
    X = (rng.standard_normal((IMAGES, 3, 30, 30)) * (2.0 ** 40 if low else 1.0)).astype(np.float32)
    err = np.abs(_run(L, geom, X) - _sums(W, X))
    assert (err <= 4 * 2.0 ** -24 * _sums(np.abs(W), np.abs(X))).all()
    L.free()


@pytest.mark.parametrize("bad", [np.inf, -np.inf])
def test_infinity_meets_bf16_weights(bad):
    """Weights that are bf16 values themselves (powers of two: nothing is left for their second and third
    term) keep an infinity's sign, and a weight of zero makes it NaN, as in fp32."""
    rng = np.random.default_rng(9)
    cb = np.array([0] + [s * 2.0 ** k for k in range(-64, 63) for s in (-1, 1)] + [1.5], np.float32)
    geom = _geom(2, 30, 1, 64)
    W = (cb[rng.integers(1, 256, (64, 2))] * (rng.random((64, 2)) < 0.7)).astype(np.float32)
    L = cl.compress_layer(W, 8, 8, 128, 128, codebook=cb, upload=True)
    assert np.array_equal(cl.decode_layer(L)[3].cpu().numpy(), W)
    X = rng.standard_normal((IMAGES, 2, 30, 30)).astype(np.float32)
    X[5, 1, 3, 4] = bad
    with np.errstate(invalid="ignore"):
        want = np.float32(bad) * W[:, 1]
    assert np.array_equal(_run(L, geom, X)[5, :, 3, 4], want.astype(np.float64), equal_nan=True)
    L.free()
