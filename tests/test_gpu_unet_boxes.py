"""The box kernels of the network's own layers against the FP64 layer oracle.

3x3x3 convolutions of a multiple of 32 input channels run from boxes of
positions in LDS (forward, data gradient), weight gradients of a multiple of
32 output channels from boxes of 256, and the transposed convolution's
parities as one-tap products.  Sizes where they can go wrong: grids smaller
than a box and one cell longer, both arrangements of positions along y and z
(16 x 1 and 8 x 2), one, two and several slabs of input channels, output
channels that fill no tile, channel slices, accumulation, enough boxes for
several splits and for the widest tiles, and odd counts in the sums.

Bars as in test_gpu_unet.py: 2e-5 of the largest reference magnitude for FP32
outputs (FP32 accumulation over at most a few thousand products), plus one
BF16 rounding (2^-8) for BF16 ones."""

import math

import numpy as np
import pytest
import torch

from gpu_common import DEV, announce, requires_gpu
from oracle import unet as O
from test_gpu_unet import NEG3, TAPS3, UP8, _bf, _check, _dev_bf, _dev_f, _host, _wide

pytestmark = [pytest.mark.gpu, requires_gpu]

SHAPES = [(1, 1, 1, 1), (2, 4, 16, 8), (1, 5, 17, 9), (1, 9, 7, 3), (2, 3, 8, 18), (1, 20, 18, 24)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cin,cout", [(32, 32), (64, 20), (32, 4), (96, 100)])
def test_conv3_boxes_forward(shape, cin, cout):
    from paper_2311_16935_amd import unet as U

    announce("conv3 boxes", shape, cin, cout)
    rng = np.random.default_rng(cin + cout + shape[1])
    x = _bf(rng.normal(size=shape + (cin,)))
    W = _bf(rng.normal(size=(27, cin, cout)) / math.sqrt(27 * cin))
    b = rng.normal(size=cout).astype(np.float32).astype(np.float64)
    xd, wd, bd = _dev_bf(_wide(x, 8, 24)), _dev_bf(W.transpose(0, 2, 1)), _dev_f(b)
    ref = O.conv3(x, W, b, relu=True)
    for off in (4, 3):  # four channels per store, and one
        y = torch.zeros(shape + (cout + 8,), dtype=torch.bfloat16, device=DEV)
        U.pu_conv(U.tensor(xd, 8, cin), wd, 27, TAPS3, bd, U.tensor(y, off, cout), shape[1:], relu=True)
        yh = _host(y)
        _check(yh[..., off:off + cout], ref, True, f"conv off={off}")
        assert np.all(yh[..., :off] == 0) and np.all(yh[..., off + cout:] == 0)
    # taps in another order, FP32 output and accumulation
    perm = rng.permutation(27)
    wp = _dev_bf(W.transpose(0, 2, 1)[perm])
    y32 = torch.zeros(shape + (cout,), dtype=torch.float32, device=DEV)
    for k in (1, 2):
        U.pu_conv(U.tensor(xd, 8, cin), wp, 27, [TAPS3[i] for i in perm], None, U.tensor(y32), shape[1:], y_fp32=True,
                  accumulate=True)
        _check(_host(y32), k * O.conv3(x, W, np.zeros(cout)), False, f"conv accumulate {k}")
    torch.cuda.synchronize()


def test_conv3_boxes_wide_tiles():
    """Enough workgroups for eight tiles along x and 64 output channels each."""
    from paper_2311_16935_amd import unet as U

    announce("conv3 wide tiles")
    rng = np.random.default_rng(5)
    for shape, cin, cout in (((1, 40, 40, 72), 32, 33), ((2, 26, 33, 64), 64, 72), ((1, 61, 8, 40), 32, 64)):
        x = _bf(rng.normal(size=shape + (cin,)))
        W = _bf(rng.normal(size=(27, cin, cout)) / math.sqrt(27 * cin))
        xd, wd = _dev_bf(x), _dev_bf(W.transpose(0, 2, 1))
        y = torch.zeros(shape + (cout,), dtype=torch.bfloat16, device=DEV)
        U.pu_conv(U.tensor(xd), wd, 27, TAPS3, None, U.tensor(y), shape[1:])
        _check(_host(y), O.conv3(x, W, np.zeros(cout)), True, f"conv {shape}")
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("cin,cout", [(32, 32), (4, 32), (20, 64), (96, 32)])
def test_conv3_boxes_backward(shape, cin, cout):
    from paper_2311_16935_amd import unet as U

    announce("conv3 boxes bwd", shape, cin, cout)
    rng = np.random.default_rng(100 + cin + shape[2])
    x = _bf(rng.normal(size=shape + (cin,)))
    W = _bf(rng.normal(size=(27, cin, cout)) / math.sqrt(27 * cin))
    gy = _bf(rng.normal(size=shape + (cout,)))
    rgx, rgW, rgb = O.conv3_backward(x, W, gy)
    xd, wd, gyd = _dev_bf(_wide(x, 8, 16)), _dev_bf(W), _dev_bf(_wide(gy, 8, 8))
    gx = torch.zeros(shape + (cin,), dtype=torch.float32, device=DEV)
    U.pu_conv(U.tensor(gyd, 8, cout), wd, 27, NEG3, None, U.tensor(gx), shape[1:], y_fp32=True)
    _check(_host(gx), rgx, False, "dgrad")
    work = torch.zeros(U.pu_wgrad_work_floats(27, cin, cout, math.prod(shape)), dtype=torch.float32, device=DEV)
    dW = torch.zeros((27, cin, cout), dtype=torch.float32, device=DEV)
    db = torch.zeros(cout, dtype=torch.float32, device=DEV)
    U.pu_conv_wgrad(U.tensor(xd, 8, cin), U.tensor(gyd, 8, cout), 27, TAPS3, dW, db, shape[1:], 1, 1, (0, 0, 0), work)
    _check(_host(dW), rgW, False, "wgrad")
    _check(_host(db), rgb, False, "bias grad")
    dW.zero_()
    U.pu_conv_wgrad(U.tensor(xd, 8, cin), U.tensor(gyd, 8, cout), 27, TAPS3, dW, None, shape[1:], 1, 1, (0, 0, 0), work)
    _check(_host(dW), rgW, False, "wgrad without bias")
    torch.cuda.synchronize()


@pytest.mark.parametrize("cin,cout", [(32, 36), (64, 32), (128, 64), (256, 128), (96, 32)])
def test_upconv_parities(cin, cout):
    """One-tap products into a channel slice (96 input channels: the general kernel)."""
    from paper_2311_16935_amd import unet as U

    announce("upconv parities", cin, cout)
    rng = np.random.default_rng(cin)
    shape, fine = (2, 3, 5, 7), (2, 6, 10, 14)
    x = _bf(rng.normal(size=shape + (cin,)))
    W = _bf(rng.normal(size=(8, cin, cout)) / math.sqrt(cin))
    xd, wt = _dev_bf(_wide(x, 8, 8)), _dev_bf(W.transpose(0, 2, 1))
    y = torch.zeros(fine + (cout + 8,), dtype=torch.bfloat16, device=DEV)
    for q, oo in enumerate(UP8):
        U.pu_conv(U.tensor(xd, 8, cin), wt[q], 1, [(0, 0, 0)], None, U.tensor(y, 4, cout), shape[1:], 1, 2, oo)
    yh = _host(y)
    _check(yh[..., 4:4 + cout], O.upconv(x, W, np.zeros(cout)), True, "upconv")
    assert np.all(yh[..., :4] == 0) and np.all(yh[..., 4 + cout:] == 0)


@pytest.mark.parametrize("c,off", [(32, 0), (32, 8), (24, 4), (7, 0)])
def test_relu_backward_widths(c, off):
    from paper_2311_16935_amd import unet as U

    announce("relu backward", c, off)
    rng = np.random.default_rng(c)
    y, g = _bf(rng.normal(size=(2, 3, 5, 4, c))), _bf(rng.normal(size=(2, 3, 5, 4, c)))
    yd, gd = _dev_bf(_wide(y, off, 8)), _dev_bf(_wide(g, 0, 8))
    U.pu_relu_backward(U.tensor(yd, off, c), U.tensor(gd, 0, c))
    assert np.array_equal(_host(gd), _wide(np.where(y > 0, g, 0.0), 0, 8))
