"""The pointwise kernel on 1x1 layers of up to 64 pixels, at the sizes where its tiles, windows of output channels
and steps end, against the oracle (needs a GPU)."""
import numpy as np
import pytest

import oracle
import paper_2407_09453_amd as bsp
from synthetic import draw_layer

from gpu_util import assert_close, kernels_of, make_layer, to_device, to_host

pytestmark = pytest.mark.gpu

# B, L, J, I, O, stride
SHAPES = [
    (1, 1, 1, 16, 8, 1),            # one pixel, half a strip
    (17, 1, 1, 32, 72, 1),          # one pixel past a tile, a window that is not full
    (64, 1, 1, 512, 24, 1),         # fewer strips than a window
    (1, 7, 7, 512, 136, 1),
    (3, 8, 8, 40, 1000, 2),         # strided, ragged last step and window
    (5, 1, 1, 256, 4096, 1),        # several workgroups share the pixels
    (63, 1, 1, 64, 16, 1),
]


def _infinities(c, n):
    """Puts an infinity of either sign and a NaN into c.X; what becomes of each output, and the input without them."""
    conv = lambda X: oracle.conv2d(X, c.W, None, c.gamma, c.bo, c.bi, c.stride, c.pad)
    rng = np.random.default_rng(n)
    hit, X0, s = {}, c.X.copy(), c.stride[0]
    for v in (np.inf, -np.inf, np.nan):
        one = np.zeros_like(c.X)
        at = rng.integers(c.X.shape[0]), rng.integers(c.M) * s, rng.integers(c.N) * s, rng.integers(c.X.shape[3])
        one[at], X0[at], c.X[at] = 1.0, 0.0, v
        hit[str(v)] = conv(one)
    up = (hit["inf"] > 0) | (hit["-inf"] < 0)
    down = (hit["inf"] < 0) | (hit["-inf"] > 0)
    nan = (hit["nan"] != 0) | (up & down)
    return up & ~nan, down & ~nan, nan, X0


def _check(n, c, kernel):
    import torch
    bo, bi = c.bo, c.bi
    layer, X = make_layer(c), to_device(c)
    Y = torch.full((c.B, c.M, c.N, c.O), float("nan"), device="cuda", dtype=torch.bfloat16)
    ran = kernels_of(lambda: layer.conv2d(X, c.stride, c.pad, out=Y))
    assert any(kernel in k for k in ran), ran
    want = oracle.conv2d(c.X, c.W, c.bias, c.gamma, bo, bi, c.stride, c.pad)
    assert_close(to_host(Y), want, "bf16", f"shape {n}")
    # bit for bit the plain call followed by torch's add and relu, each rounding once
    R = torch.randn(Y.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(n)).bfloat16()
    post = lambda y: torch.relu(y.float() + R.float()).bfloat16()
    assert torch.equal(layer.conv2d(X, c.stride, c.pad, residual=R, relu=True), post(Y)), n
    # an infinity reaches the rows that keep its channel and no others
    up, down, nan, X0 = _infinities(c, n)
    Y1 = layer.conv2d(to_device(c), c.stride, c.pad)
    y, ok = to_host(Y1), ~(up | down | nan)
    assert (np.isnan(y) == nan).all() and (np.isposinf(y) == up).all() and (np.isneginf(y) == down).all(), n
    want = oracle.conv2d(X0, c.W, c.bias, c.gamma, bo, bi, c.stride, c.pad)
    assert_close(np.where(ok, y, 0.0), np.where(ok, want, 0.0), "bf16", f"shape {n}, infinities")
    Y2 = layer.conv2d(to_device(c), c.stride, c.pad, residual=R, relu=True)
    same = torch.from_numpy(~nan).cuda()
    assert torch.equal(Y2[same], post(Y1)[same]), n


def _case(n, shape, bo, bi, density):
    B, L, J, I, O, s = shape
    print("case", n, shape, bo, bi, density, flush=True)
    return draw_layer("t", B=B, L=L, J=J, I=I, O=O, H=1, K=1, stride=(s, s), pad=(0, 0), bo=bo, bi=bi, dtype="bf16",
                      mask_kind="bernoulli", density=density, seed=9900 + n, b_std=0.5)


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("density", [0.0, 0.5, 1.0])
def test_few_pixels(bo, bi, density):
    for n, shape in enumerate(SHAPES):
        _check(n, _case(n, shape, bo, bi, density), "conv_pw")


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("n,tiles,steps", [(0, 2, 2), (1, 2, 4), (2, 2, 8), (3, 4, 2), (4, 4, 4), (5, 4, 8)])
def test_lane_tiles_and_steps(bo, bi, n, tiles, steps):
    """Layers of many channels out, whose workgroups have several lane tiles a wave, with as many registers for weights
    as a strip's steps need."""
    shape = [(33, 1, 1, 40, 5200, 1), (6, 3, 9, 112, 5208, 2), (64, 1, 1, 512, 6000, 1), (5, 1, 1, 40, 10400, 1), (33, 1, 1, 112, 10408, 1),
             (1, 7, 7, 256, 12000, 1)][n]
    _check(n, _case(20 + n, shape, bo, bi, 0.5), "conv_pw<%d, %d, %d," % (tiles, 4 if bi == 4 else 8, steps))


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
def test_few_pixels_int8_bit_exact(bo, bi):
    import torch
    for n, (B, L, J, I, O, s) in enumerate([(1, 1, 1, 16, 16, 1), (17, 1, 1, 80, 80, 1), (64, 1, 1, 1024, 48, 1),
                                            (3, 8, 8, 208, 1008, 2), (1, 7, 7, 512, 272, 1), (49, 1, 1, 2048, 4096, 1)]):
        rng = np.random.default_rng(9950 + n)
        X = rng.integers(-128, 128, (B, L, J, I), dtype=np.int8)
        W = rng.integers(-128, 128, (O, 1, 1, I), dtype=np.int8)
        bias = rng.integers(-2 ** 18, 2 ** 18, O).astype(np.int32)
        gamma = (rng.random((O // bo, I // bi)) < 0.5).astype(np.uint8)
        print("case", n, (B, L, J, I, O, s), bo, bi, flush=True)
        layer = bsp.BspLayerI8(W, gamma, bo, bi, bias=bias)
        Y = torch.full((B, -(-L // s), -(-J // s), O), 99, dtype=torch.int8, device="cuda")
        ran = kernels_of(lambda: layer.conv2d(torch.from_numpy(X).cuda(), (s, s), (0, 0), shift=9, out=Y))
        # (16x4 blocks of many kept channels: a strip's union may not fit the sections' limits)
        assert any("conv_pw" in k for k in ran) or (bo, I) == (16, 2048), ran
        want = oracle.conv2d_i8(X, W, bias, gamma, bo, bi, (s, s), (0, 0), shift=9)
        assert (Y.cpu().numpy() == want).all(), n
