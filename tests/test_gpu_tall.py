"""The persistent kernel for three-row windows (csrc/bsp_tall.hip) through the dispatcher, against fp64: ragged
tiles, strips that fill no group, slabs of few channels, every split of the contraction (needs a GPU)."""
import numpy as np
import pytest

import paper_2407_09453_amd as bsp

from gpu_util import conv_fp64, kernels_of

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, L, J, I, O, K, padding, blocks, density
    (16, 28, 28, 512, 512, 3, (1, 1), (8, 8), 0.5),     # whole tiles, four slabs
    (5, 45, 43, 264, 328, 3, (1, 1), (8, 8), 0.5),      # ragged rows and columns, a slab of one chunk
    (7, 25, 26, 288, 520, 3, (0, 0), (8, 8), 0.75),     # no padding; the contraction in two shares
    (2, 79, 89, 104, 296, 3, (1, 1), (8, 8), 0.5),      # nineteen strips, one slab
    (3, 66, 75, 72, 344, 3, (1, 1), (16, 4), 0.75),     # units of four channels
    (60, 25, 13, 424, 296, 3, (1, 1), (16, 4), 0.5),
    (2, 65, 65, 592, 152, 3, (1, 1), (4, 16), 0.75),    # results in pieces of eight bytes; four shares
    (16, 13, 41, 384, 88, 5, (1, 2), (8, 8), 0.5),      # 3x5; four shares of tiles two columns wide
    (10, 106, 10, 144, 472, 3, (1, 1), (8, 8), 0.75),   # three bands in a tile
    (29, 21, 21, 88, 264, 3, (1, 1), (16, 4), 0.75),    # two column groups
    (17, 19, 19, 80, 376, 3, (1, 1), (8, 8), 1.0),      # two of each
    (6, 103, 41, 192, 400, 1, (1, 0), (4, 16), 0.5),    # 3x1
    # several items to a workgroup, one after the other, and several images to a tile
    (160, 10, 6, 224, 608, 3, (1, 1), (8, 8), 1.0),     # both
    (200, 9, 8, 256, 608, 1, (1, 0), (16, 4), 1.0),
    (200, 10, 6, 96, 296, 3, (1, 1), (4, 16), 0.25),    # and two shares of the contraction
    (200, 8, 6, 512, 344, 3, (1, 1), (16, 4), 0.25),
    (160, 8, 9, 288, 200, 5, (1, 2), (4, 16), 0.75),    # items and shares, fourteen rows
    (33, 20, 25, 384, 296, 3, (1, 1), (8, 8), 0.5),     # seven rows
    (5, 42, 48, 384, 608, 3, (1, 1), (16, 4), 1.0),
    (160, 7, 8, 512, 200, 1, (1, 0), (4, 16), 0.75),    # images and shares
    (160, 9, 6, 136, 72, 3, (1, 1), (8, 8), 0.5),       # four shares
    (100, 10, 8, 96, 152, 5, (1, 2), (16, 4), 1.0),
    (2, 56, 66, 384, 152, 3, (1, 1), (8, 8), 1.0),
    (200, 7, 5, 72, 512, 3, (1, 1), (4, 16), 0.5),      # six images
    (100, 10, 9, 104, 296, 3, (1, 1), (8, 8), 0.75),    # three images, two column groups
]


@pytest.mark.parametrize("n", range(len(SHAPES)))
def test_tall_kernel(n):
    import torch
    B, L, J, I, O, K, pad, (bo, bi), density = SHAPES[n]
    print("tall case", n, SHAPES[n], flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    rng = np.random.default_rng(n)
    gamma = (rng.random((-(-O // bo), -(-I // bi))) < density).astype(np.uint8)
    gamma[1] = 0                     # a block row with nothing
    gamma[2:4, : gamma.shape[1] // 2] = 0
    keep = torch.from_numpy(np.kron(gamma, np.ones((bo, bi), np.uint8))[:O, :I].copy()).cuda()[:, None, None, :]
    X = torch.randn(B, L, J, I, generator=gen, device="cuda").bfloat16()
    W = (torch.randn(O, 3, K, I, generator=gen, device="cuda") * (2.0 / (density * I * 3 * K)) ** 0.5).bfloat16()
    bias = rng.standard_normal(O).astype(np.float32)
    layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, bo, bi, "bf16", bias=bias)
    shape = layer.out_shape(B, L, J, (1, 1), pad)
    out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (1, 1), pad, out=out))
    assert any("conv_tall" in k for k in ran), ran
    want = conv_fp64(X, W * keep, 1, pad) + torch.from_numpy(bias).cuda()
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 6e-3 * scale).all())   # one rounding to bf16 is 3.9e-3 at most
    # the fused epilogue: the same sums, then torch's own arithmetic in bf16
    R = torch.randn(shape, generator=gen, device="cuda").bfloat16()
    fused = layer.conv2d(X, (1, 1), pad, residual=R, relu=True)
    assert torch.equal(fused, torch.relu(out + R))
    assert torch.equal(layer.conv2d(X, (1, 1), pad, relu=True), torch.relu(out))
