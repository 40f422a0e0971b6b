"""An infinite activation reaches the weight gradients of the taps that see
its cell, and no others: the kernels' tiles hold positions past the grid's end,
where the gradient is 0 and an infinity inside the grid must not be multiplied
by it.  Grids that fill their boxes of positions and grids that end inside one,
along every axis and for both arrangements of positions (16 x 2 and 8 x 4
along y and z), the infinity in every corner and in the middle.

The expected values: the FP64 oracle's, with the cell set to 0, and infinity
with the sign of the gradient where a tap sees the cell.  Bar for the finite
ones as in test_gpu_unet.py (2e-5 of the largest reference magnitude)."""

import itertools
import math

import numpy as np
import pytest
import torch

from gpu_common import DEV, announce, requires_gpu
from oracle import unet as O
from test_gpu_unet import TAPS3, _bf, _check, _dev_bf, _host

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shape", [(1, 4, 16, 8), (1, 5, 17, 9), (2, 9, 7, 3), (1, 20, 33, 26), (1, 23, 24, 31)])
@pytest.mark.parametrize("cin,cout", [(32, 32), (4, 64)])
def test_infinite_activation_stays_with_the_taps_that_see_it(shape, cin, cout):
    from paper_2311_16935_amd import unet as U

    announce("wgrad of an infinity", shape, cin, cout)
    rng = np.random.default_rng(shape[3] + cin)
    n, d, h, w = shape
    x = _bf(rng.normal(size=shape + (cin,)))
    gy = _bf(rng.normal(size=shape + (cout,)))
    gyd = _dev_bf(gy)
    work = torch.zeros(U.pu_wgrad_work_floats(27, cin, cout, math.prod(shape)), dtype=torch.float32, device=DEV)
    dW = torch.zeros((27, cin, cout), dtype=torch.float32, device=DEV)
    db = torch.zeros(cout, dtype=torch.float32, device=DEV)
    cells = list(itertools.product((0, d - 1), (0, h - 1), (0, w - 1))) + [(d // 2, h // 2, w // 2)]
    for k, (z, y, xx) in enumerate(cells):
        b, c = k % n, k % cin
        xi = x.copy()
        xi[b, z, y, xx, c] = 0.0
        _, ref, rb = O.conv3_backward(xi, np.zeros((27, cin, cout)), gy)
        xi[b, z, y, xx, c] = np.inf
        U.pu_conv_wgrad(U.tensor(_dev_bf(xi)), U.tensor(gyd), 27, TAPS3, dW, db, shape[1:], 1, 1, (0, 0, 0), work)
        got = _host(dW)
        for t, (dz, dy, dx) in enumerate(TAPS3):
            pz, py, px = z - dz, y - dy, xx - dx
            if 0 <= pz < d and 0 <= py < h and 0 <= px < w:
                assert np.array_equal(got[t, c], np.sign(gy[b, pz, py, px]) * np.inf), (k, t)
                got[t, c] = ref[t, c]
        _check(got, ref, False, f"cell {k}")
        _check(_host(db), rb, False, f"bias, cell {k}")
