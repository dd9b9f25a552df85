"""The pointwise kernel on int8 codes, bit for bit against the integer oracle, at the sizes where its
tiles, windows of output channels and steps end (needs a GPU)."""
import numpy as np
import pytest

import oracle
import paper_2407_09453_amd as bsp

pytestmark = pytest.mark.gpu

# B, L, J, I, O, stride
SHAPES = [
    (1, 5, 13, 16, 16, 1),          # one pixel past 64, one unit, one strip
    (1, 9, 9, 80, 80, 1),           # a window of output channels that is not full
    (2, 17, 17, 208, 48, 1),        # fewer strips than a window, ragged last step
    (3, 14, 14, 256, 144, 2),       # strided
    (8, 28, 28, 64, 272, 1),        # thin tile, many pixels, ragged last window
    (1, 12, 12, 4096, 32, 1),       # the most channels one slab holds
    (40, 40, 40, 32, 64, 1),        # enough pixels for the small groups of strips
]


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("density", [0.4, 1.0])
def test_pointwise_int8_bit_exact(bo, bi, density):
    import torch
    for n, (B, L, J, I, O, s) in enumerate(SHAPES):
        rng = np.random.default_rng(9600 + n)
        X = rng.integers(-128, 128, (B, L, J, I), dtype=np.int8)
        W = rng.integers(-128, 128, (O, 1, 1, I), dtype=np.int8)
        bias = rng.integers(-2 ** 18, 2 ** 18, O).astype(np.int32)
        bias[0], bias[-1] = 2 ** 31 - 1, -2 ** 31            # the sum and bias leave 32 bits
        gamma = (rng.random((O // bo, I // bi)) < density).astype(np.uint8)
        print("case", n, SHAPES[n], bo, bi, flush=True)
        layer = bsp.BspLayerI8(W, gamma, bo, bi, bias=bias)
        sums = oracle.conv2d_i8(X, W, np.zeros(O, np.int32), gamma, bo, bi, (s, s), (0, 0)).astype(np.int64) + bias
        for shift in (0, 9, 24, 25, 31):
            Y = torch.full(sums.shape, 99, dtype=torch.int8, device="cuda")
            layer.conv2d(torch.from_numpy(X).cuda(), (s, s), (0, 0), shift=shift, out=Y)
            torch.cuda.synchronize()
            want = np.clip((sums + (1 << shift >> 1)) >> shift, -128, 127)
            assert (Y.cpu().numpy() == want).all(), (n, shift)
