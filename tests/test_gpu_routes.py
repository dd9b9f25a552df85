"""Layers on either side of the dispatcher's lines: the kernel that runs, and its results against fp64
(needs a GPU)."""
import numpy as np
import pytest

import paper_2407_09453_amd as bsp

from gpu_util import conv_fp64, kernels_of

pytestmark = pytest.mark.gpu


def _draw(n, B, L, J, I, O, H, K, bo, bi):
    import torch
    gen = torch.Generator("cuda").manual_seed(n)
    gamma = (np.random.default_rng(n).random((-(-O // bo), -(-I // bi))) < 0.5).astype(np.uint8)
    gamma[0, 0] = 1
    keep = torch.from_numpy(np.kron(gamma, np.ones((bo, bi), np.uint8))[:O, :I].copy()).cuda()
    X = torch.randn(B, L, J, I, generator=gen, device="cuda")
    W = torch.randn(O, H, K, I, generator=gen, device="cuda") * (2.0 / (I * H * K)) ** 0.5
    return X, W, gamma, keep[:, None, None, :]


BF16 = [
    # B, L, J, I, O, H, K, stride, blocks, kernel
    (16, 17, 17, 160, 192, 1, 7, 1, (8, 8), "conv_any"), (4, 57, 57, 272, 192, 1, 7, 1, (8, 8), "conv_rows"),
    (28, 37, 37, 32, 184, 1, 7, 1, (4, 16), "conv_lds"), (8, 22, 22, 192, 104, 7, 1, 1, (4, 16), "conv_any"),
    (1, 56, 56, 64, 64, 3, 3, 1, (8, 8), "conv_any"), (4, 35, 35, 64, 96, 3, 3, 1, (8, 8), "conv_band"),
    (21, 77, 77, 8, 160, 3, 3, 2, (4, 16), "conv_lds"), (40, 34, 11, 168, 24, 3, 5, 1, (4, 16), "conv_rows"),
    (15, 18, 10, 288, 112, 7, 7, 1, (4, 16), "conv_rows"), (5, 73, 73, 24, 32, 5, 5, 1, (4, 16), "conv_lds"),
    (27, 37, 8, 64, 144, 7, 7, 1, (8, 8), "conv_tile"), (3, 25, 25, 248, 16, 5, 5, 1, (4, 16), "conv_any"),
    (33, 1, 1, 2048, 4096, 1, 1, 1, (4, 16), "fc_stream"), (64, 1, 1, 2048, 1000, 1, 1, 1, (8, 8), "conv_any"),
]


@pytest.mark.parametrize("n", range(len(BF16)))
def test_bf16_layers(n):
    import torch
    B, L, J, I, O, H, K, s, (bo, bi), kernel = BF16[n]
    X, W, gamma, keep = _draw(n, B, L, J, I, O, H, K, bo, bi)
    X, W = X.bfloat16(), W.bfloat16()
    bias = np.random.default_rng(n).standard_normal(O).astype(np.float32)
    layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, bo, bi, "bf16", bias=bias)
    pad = (H // 2, K // 2)
    out = torch.full(layer.out_shape(B, L, J, (s, s), pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (s, s), pad, out=out))
    assert any(kernel in k for k in ran), ran
    want = conv_fp64(X, W * keep, s, pad) + torch.from_numpy(bias).cuda()
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 6e-3 * scale).all())   # one rounding to bf16 is 3.9e-3 at most


@pytest.mark.parametrize("B,L,J,I,O,H,K,stride,any_shape", [
    (16, 17, 17, 192, 320, 3, 3, 2, True), (32, 35, 35, 288, 384, 3, 3, 2, False),     # 3x3 strided: 66 K, some 400 K
    (16, 8, 8, 448, 384, 3, 3, 1, True), (22, 14, 14, 168, 320, 3, 3, 1, False),       # a third of the channels in: 155 K, 205 K
    (8, 7, 7, 512, 512, 3, 3, 1, True), (5, 10, 10, 512, 512, 3, 3, 1, False), (8, 14, 14, 512, 512, 3, 3, 2, False),  # many weights
    (1, 58, 58, 584, 32, 3, 3, 1, True), (4, 50, 50, 232, 80, 3, 3, 1, False),         # few strips, and too many pixels
    (16, 8, 8, 384, 384, 3, 1, 1, True), (21, 32, 32, 496, 56, 3, 1, 1, False), (4, 20, 20, 200, 104, 3, 1, 2, True),
    (16, 8, 8, 448, 384, 1, 3, 1, True), (30, 32, 32, 320, 192, 1, 3, 1, False),
])
def test_any_shape_or_row_bands(B, L, J, I, O, H, K, stride, any_shape):
    """Either side of the lines between the any-shape and the row-band kernel (or the one that goes before it)."""
    import torch
    X, W, gamma, keep = _draw(I + O, B, L, J, I, O, H, K, 8, 8)
    X, W, pad = X.bfloat16(), W.bfloat16(), (H // 2, K // 2)
    layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, 8, 8, "bf16")
    out = torch.full(layer.out_shape(B, L, J, (stride, stride), pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (stride, stride), pad, out=out))
    assert any("conv_any" in k for k in ran) == any_shape, ran
    want = conv_fp64(X, W * keep, stride, pad)
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 6e-3 * scale).all())   # one rounding to bf16 is 3.9e-3 at most


@pytest.mark.parametrize("B,L,I,O,H,K,stride,least,most,any_shape", [
    (4, 24, 360, 264, 1, 7, 1, 120000, 200000, True), (7, 24, 360, 264, 1, 7, 1, 200000, 300000, False),
    (4, 35, 488, 88, 3, 1, 1, 45000, 80000, True), (18, 28, 216, 64, 3, 1, 1, 45000, 80000, False),     # up to 5000 pixels, and more
    (28, 30, 360, 256, 3, 1, 2, 45000, 340000, True),
    (7, 48, 280, 88, 3, 3, 2, 60000, 300000, True), (2, 56, 416, 56, 3, 3, 2, 30000, 60000, True), (20, 47, 416, 40, 3, 3, 2, 60000, 300000, False),
    (5, 16, 488, 176, 3, 3, 1, 30000, 115000, True), (8, 14, 256, 256, 3, 3, 1, 30000, 115000, False),  # by the kernels' models
    (14, 8, 448, 384, 3, 3, 1, 115000, 200000, True), (16, 14, 256, 256, 3, 3, 1, 115000, 300000, False),  # few pixels, and more
])
def test_lines_to_the_row_band_kernel(B, L, I, O, H, K, stride, least, most, any_shape):
    """Layers inside each band of matrix instructions that bsp_rules.h gives the any-shape or the row-band kernel (or the one before it)."""
    import torch
    X, W, gamma, keep = _draw(I + O, B, L, L, I, O, H, K, 8, 8)
    X, W, pad = X.bfloat16(), W.bfloat16(), (H // 2, K // 2)
    layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, 8, 8, "bf16")
    out = torch.full(layer.out_shape(B, L, L, (stride, stride), pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    mm = -(-out.numel() // O // 16) * int(layer.plan[18])  # steps of all strips
    assert least < mm <= most, mm
    ran = kernels_of(lambda: layer.conv2d(X, (stride, stride), pad, out=out))
    assert any("conv_any" in k for k in ran) == any_shape, ran
    want = conv_fp64(X, W * keep, stride, pad)
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 6e-3 * scale).all())   # one rounding to bf16 is 3.9e-3 at most


F32 = [
    (34, 15, 15, 5, 125, 1, 1, 1, (16, 4), "conv_general"), (25, 49, 49, 79, 180, 1, 1, 1, (16, 4), "conv_f32<"),
    (6, 14, 14, 11, 118, 1, 1, 1, (8, 8), "conv_general"), (4, 13, 21, 64, 102, 1, 3, 1, (8, 8), "conv_f32x3<"),
    (50, 50, 12, 3, 323, 3, 3, 1, (16, 4), "conv_general"), (8, 43, 43, 1, 496, 5, 5, 1, (16, 4), "conv_f32<"),
    (192, 1, 1, 5, 110, 1, 1, 1, (16, 4), "conv_general"), (192, 1, 1, 9, 110, 1, 1, 1, (16, 4), "fc_f32<"),
    (5, 20, 20, 30, 33, 1, 1, 2, (4, 16), "conv_general"), (5, 20, 20, 130, 33, 1, 1, 2, (4, 16), "conv_f32<"),
    # whole chunks of channels: on either side of the three-part kernel's line
    (4, 13, 21, 60, 102, 1, 3, 1, (8, 8), "conv_f32<"), (5, 70, 70, 8, 768, 1, 1, 1, (8, 8), "conv_general"),
    (256, 1, 1, 512, 104, 1, 1, 1, (8, 8), "fc_f32<"), (257, 1, 1, 512, 104, 1, 1, 1, (8, 8), "conv_f32x3<"),
    (2, 18, 105, 1400, 16, 1, 1, 1, (8, 8), "conv_f32<"), (2, 18, 105, 1400, 24, 1, 1, 1, (8, 8), "conv_f32x3<"),
    (2, 32, 10, 400, 72, 3, 3, 1, (4, 16), "conv_f32<"), (7, 32, 10, 400, 72, 3, 3, 1, (4, 16), "conv_f32x3<"),
    (6, 15, 15, 504, 109, 5, 5, 2, (8, 8), "conv_f32<"), (24, 15, 15, 504, 109, 5, 5, 2, (8, 8), "conv_f32x3<"),
    (2, 9, 10, 2048, 512, 3, 3, 1, (8, 8), "conv_f32<"),
]


@pytest.mark.parametrize("n", range(len(F32)))
def test_f32_layers(n):
    import torch
    B, L, J, I, O, H, K, s, (bo, bi), kernel = F32[n]
    X, W, gamma, keep = _draw(100 + n, B, L, J, I, O, H, K, bo, bi)
    bias = np.random.default_rng(n).standard_normal(O).astype(np.float32)
    layer = bsp.BspLayer(W.cpu().numpy(), gamma, bo, bi, "f32", bias=bias)
    pad = (H // 2, K // 2)
    out = torch.full(layer.out_shape(B, L, J, (s, s), pad), float("nan"), device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (s, s), pad, out=out))
    assert any(kernel in k for k in ran), ran
    want = conv_fp64(X, W * keep, s, pad) + torch.from_numpy(bias).cuda()
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    # eight standard deviations of a sum of n products in fp32, sqrt(n / 6) * 2^-24 (up to 700 terms: 1e-5)
    assert bool(((out.double() - want).abs() <= max(1e-5, 8 * (0.6 * I * H * K / 6) ** 0.5 * 2.0 ** -24) * scale).all())


def _i8_layer(n, B, L, J, I, O, H, K, bo, bi):
    """A layer of codes and its exact sums (fp64 holds them)."""
    import torch
    gen = torch.Generator("cuda").manual_seed(n)
    X, _, gamma, keep = _draw(n, 1, 1, 1, I, O, 1, 1, bo, bi)
    X = torch.randint(-128, 128, (B, L, J, I), generator=gen, device="cuda", dtype=torch.int8)
    W = torch.randint(-128, 128, (O, H, K, I), generator=gen, device="cuda", dtype=torch.int8)
    bias = np.random.default_rng(n).integers(-40000, 40000, O, dtype=np.int32)
    return bsp.BspLayerI8(W.cpu().numpy(), gamma, bo, bi, bias=bias), X, W * keep, torch.from_numpy(bias).cuda()


def _rescale(acc, shift):
    import torch
    return ((acc + ((1 << shift) >> 1)) >> shift).clamp(-128, 127).to(torch.int8)


I8 = [
    # B, L, J, I, O, H, K, stride, blocks, 8-bit results, kernel
    (11, 23, 26, 24, 40, 1, 1, 1, (16, 4), True, "conv_general"), (11, 23, 26, 22, 40, 1, 1, 1, (16, 4), True, "conv_any"),
    (9, 28, 30, 16, 16, 1, 1, 1, (4, 16), False, "conv_general"), (9, 28, 30, 40, 16, 1, 1, 1, (8, 8), False, "conv_any"),
    (25, 39, 41, 32, 32, 1, 1, 1, (8, 8), False, "conv_any"), (25, 39, 41, 16, 80, 1, 1, 2, (16, 4), False, "conv_general"),
    (25, 79, 41, 16, 112, 1, 1, 1, (8, 8), False, "conv_general"), (25, 79, 41, 24, 112, 1, 1, 1, (8, 8), False, "conv_any"),
    (1, 330, 331, 640, 32, 1, 1, 1, (8, 8), True, "conv_lds"), (1, 330, 331, 640, 48, 1, 1, 1, (8, 8), True, "conv_any"),
    (16, 37, 38, 144, 80, 1, 3, 1, (4, 16), True, "conv_any"), (35, 37, 37, 176, 160, 1, 5, 1, (4, 16), True, "conv_any"),
    (32, 7, 7, 512, 512, 3, 3, 1, (8, 8), True, "conv_any"), (50, 32, 32, 192, 64, 3, 3, 1, (8, 8), True, "conv_any"),
]


@pytest.mark.parametrize("n", range(len(I8)))
def test_i8_layers(n):
    import torch
    B, L, J, I, O, H, K, s, (bo, bi), y8, kernel = I8[n]
    layer, X, W, bias = _i8_layer(200 + n, B, L, J, I, O, H, K, bo, bi)
    pad = (H // 2, K // 2)
    dt = torch.int8 if y8 else torch.int32
    out = torch.full(layer.out_shape(B, L, J, (s, s), pad), 77, dtype=dt, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (s, s), pad, shift=9 if y8 else None, out=out))
    assert any(kernel in k for k in ran), ran
    acc = conv_fp64(X, W, s, pad).to(torch.int64) + bias
    assert torch.equal(out, _rescale(acc, 9) if y8 else acc.int())


def test_i8_activations_beyond_the_any_shape_kernels_reach():
    """Between 2 and 4 GiB of a pointwise layer's codes, several slabs: the LDS-resident kernel takes them."""
    import torch
    B, L, I, O = 53, 252, 640, 48
    layer, X, W, bias = _i8_layer(300, B, L, L, I, O, 1, 1, 8, 8)
    out = torch.full((B, L, L, O), 77, dtype=torch.int8, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, shift=9, out=out))
    assert X.numel() >= 1 << 31 and any("conv_lds" in k for k in ran), ran
    for b in (0, B // 2, B - 1):
        assert torch.equal(out[b:b + 1], _rescale(conv_fp64(X[b:b + 1], W, 1, (0, 0)).to(torch.int64) + bias, 9))


@pytest.mark.parametrize("O", (16, 32, 48, 64))
@pytest.mark.parametrize("I", (144, 272, 640, 1008))
@pytest.mark.parametrize("B,L", ((2, 57), (29, 56)))
def test_i8_pointwise_layers_of_few_strips(B, L, I, O):
    """Every lane tile that the pointwise kernel's choice ends at, pixels that do not fill the last one."""
    import torch
    bo, bi = ((8, 8), (4, 16), (16, 4))[(O // 16 + I) % 3]
    layer, X, W, bias = _i8_layer(O + I, B, L, L - 1, I, O, 1, 1, bo, bi)
    out = torch.full((B, L, L - 1, O), 77, dtype=torch.int8, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, shift=9, out=out))
    assert any("conv_pw" in k for k in ran), ran
    assert torch.equal(out, _rescale(conv_fp64(X, W, 1, (0, 0)).to(torch.int64) + bias, 9))
