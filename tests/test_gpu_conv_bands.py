"""The 32 -> 64 channel convolution and its gradients by bands of rows in LDS,
against the float64 oracle over the same bf16 operands.  Tolerances: 2^-8 of
the value (half an ulp of bf16 is 2^-9) plus float32 accumulation error for
bf16 outputs, normwise 1e-5 for float32 ones."""
import numpy as np
import pytest
import torch

import oracle
from paper_2211_02753_amd import _lib as L

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bf16(a):
    """(device bit patterns, the float32 values they hold)"""
    r = oracle.bf16_round(np.asarray(a, np.float32))
    return torch.from_numpy((r.view(np.uint32) >> 16).astype(np.uint16).view(np.int16).copy()).to(DEV), r


def values(t):
    return (t.cpu().numpy().view(np.uint16).astype(np.uint32) << 16).view(np.float32)


def close_bf16(got, ref):
    ref = np.asarray(ref, np.float64)
    assert np.all(np.abs(got.astype(np.float64) - ref) <= 2.0 ** -8 * np.abs(ref) + 1e-4 * max(np.max(np.abs(ref)), 1e-30))


def run(x, w, dy, bias, mask, B, H, W, relu):
    lib, s = L.load(), L.stream_handle(torch.device(DEV))
    y = torch.empty((B, H - 2, W - 2, 64), dtype=torch.int16, device=DEV)
    dx = torch.empty((B, H, W, 32), dtype=torch.int16, device=DEV)
    dw = torch.empty((64, 3, 3, 32), dtype=torch.float32, device=DEV)
    db = torch.empty(64, dtype=torch.float32, device=DEV)
    L.check("fwd", lib.tdp_conv3x3_fwd_bf16(L.ptr(x), L.ptr(w), L.ptr(bias), B, H, W, 32, 64, relu, L.ptr(y), s))
    L.check("dgrad", lib.tdp_conv3x3_dgrad_bf16(L.ptr(dy), L.ptr(w), L.ptr(mask), B, H, W, 32, 64, L.ptr(dx), s))
    L.check("wgrad", lib.tdp_conv3x3_wgrad_bf16(L.ptr(x), L.ptr(dy), B, H, W, 32, 64, L.ptr(dw), L.ptr(db), s))
    return y, dx, dw, db


# one output pixel; several bands per workgroup; ragged last bands; the widest rows of each pass's bands (98 input
# columns for the input gradient, 125 for the forward, 208 for the weight gradient) and rows too wide for any
@pytest.mark.parametrize("B,H,W", [(1, 3, 3), (900, 5, 6), (3, 26, 26), (2, 33, 19), (1, 9, 96), (1, 6, 97), (2, 5, 125),
                                   (1, 5, 126), (1, 7, 208), (1, 4, 209), (1, 4, 578), (1, 3, 640)])
def test_conv_bands(B, H, W):
    rng = np.random.default_rng(B + 31 * H + W)
    xd, x = bf16(rng.standard_normal((B, H, W, 32)))
    wd, w = bf16(rng.standard_normal((64, 3, 3, 32)) * 0.1)
    dyd, dy = bf16(rng.standard_normal((B, H - 2, W - 2, 64)))
    md, m = bf16(np.maximum(rng.standard_normal((B, H, W, 32)), 0))
    bias = rng.standard_normal(64).astype(np.float32)
    print("conv bands", B, H, W, flush=True)
    y, dx, dw, db = run(xd, wd, dyd, torch.from_numpy(bias).to(DEV), md, B, H, W, 1)
    close_bf16(values(y), oracle.conv3x3_fwd(x, w, bias, relu=True))
    ref_dx = oracle.conv3x3_dgrad(dy, w, H, W)
    close_bf16(values(dx), ref_dx * (m > 0))
    rdw, rdb = oracle.conv3x3_wgrad(x, dy)
    for got, ref in ((dw, rdw), (db, rdb)):
        assert np.max(np.abs(got.cpu().numpy() - ref)) <= 1e-5 * np.max(np.abs(ref))
    y, dx, _, _ = run(xd, wd, dyd, None, None, B, H, W, 0)  # no bias, no mask, no ReLU
    close_bf16(values(y), oracle.conv3x3_fwd(x, w, np.zeros(64, np.float32), relu=False))
    close_bf16(values(dx), ref_dx)


# bands of several images: as many as fit, the last band with fewer, images of one output row or pixel, images that
# fit twice under the weight gradient's limits and not under the forward's
@pytest.mark.parametrize("B,H,W", [(5000, 3, 3), (1537, 5, 5), (1111, 8, 8), (1030, 3, 11), (1031, 9, 4), (530, 16, 16),
                                   (260, 18, 18)])
def test_conv_bands_of_small_images(B, H, W):
    test_conv_bands(B, H, W)


def test_conv_bands_keep_infinities_to_their_taps():
    """A value that is not finite reaches exactly the outputs whose taps touch it."""
    rng = np.random.default_rng(5)
    B, H, W = 2, 9, 11
    x, dy = rng.standard_normal((B, H, W, 32)), rng.standard_normal((B, H - 2, W - 2, 64))
    x[0, 0, W - 1, 3] = np.inf      # only taps with kx = 2 and ky = 0 see the corner
    x[1, 4, 0, 7] = np.nan          # only kx = 0
    dy[1, 2, W - 3, 5] = np.inf
    xd, xv = bf16(x)
    dyd, dyv = bf16(dy)
    wd, w = bf16(rng.standard_normal((64, 3, 3, 32)) * 0.1)
    y, dx, dw, db = run(xd, wd, dyd, None, None, B, H, W, 0)
    with np.errstate(invalid="ignore"):
        refs = (oracle.conv3x3_fwd(xv, w, np.zeros(64, np.float32), relu=False), oracle.conv3x3_dgrad(dyv, w, H, W),
                *oracle.conv3x3_wgrad(xv, dyv))
    for got, ref in zip((values(y), values(dx), dw.cpu().numpy(), db.cpu().numpy()), refs):
        assert np.array_equal(np.isfinite(got), np.isfinite(ref))
        assert np.array_equal(np.isnan(got), np.isnan(ref))


def test_conv_bands_keep_infinities_to_their_images():
    """Images that share a band do not see each other's values."""
    rng = np.random.default_rng(6)
    B, H, W = 2051, 4, 5
    x, dy = rng.standard_normal((B, H, W, 32)), rng.standard_normal((B, H - 2, W - 2, 64))
    x[700, H - 1, W - 1, 2], x[1401, 0, 0, 9] = np.inf, np.nan
    dy[800, H - 3, W - 3, 5] = np.inf
    xd, xv = bf16(x)
    dyd, dyv = bf16(dy)
    wd, w = bf16(rng.standard_normal((64, 3, 3, 32)) * 0.1)
    y, dx, dw, db = run(xd, wd, dyd, None, None, B, H, W, 0)
    with np.errstate(invalid="ignore"):
        refs = (oracle.conv3x3_fwd(xv, w, np.zeros(64, np.float32), relu=False), oracle.conv3x3_dgrad(dyv, w, H, W),
                *oracle.conv3x3_wgrad(xv, dyv))
    for got, ref in zip((values(y), values(dx), dw.cpu().numpy(), db.cpu().numpy()), refs):
        assert np.array_equal(np.isfinite(got), np.isfinite(ref))
        assert np.array_equal(np.isnan(got), np.isnan(ref))
