"""The kernel that streams bands past weights in registers (csrc/bsp_bands.hip) through the dispatcher: bit for bit against
the band kernel, whose steps it takes, and against fp64 where that declines.  Every instance, strips of one
to sixteen, rows and columns that fill no tile, one and two sets of buffers, infinities (needs a GPU)."""
import numpy as np
import pytest

import paper_2407_09453_amd as bsp

from gpu_util import conv_fp64, kernels_of

pytestmark = pytest.mark.gpu

CASES = [
    # B, L, J, I, O, padding, blocks, density, residual, relu, the band kernel takes it
    (16, 112, 112, 64, 64, 1, (8, 8), 0.5, True, True, True),    # four strips of five steps
    (17, 41, 43, 64, 64, 0, (8, 8), 1.0, False, True, True),     # six; rows and columns that end within a tile
    (9, 99, 51, 32, 32, 0, (8, 8), 0.5, True, False, False),     # two strips, two column tiles, one set of buffers
    (13, 99, 51, 16, 24, 1, (8, 8), 1.0, False, True, False),     # half a strip
    (31, 50, 70, 16, 16, 1, (8, 8), 1.0, True, True, False),     # one strip, four column tiles
    (18, 61, 60, 24, 48, 1, (4, 16), 0.5, False, False, False),  # three strips; a pixel of three pieces
    (11, 90, 91, 64, 72, 1, (8, 8), 0.5, True, True, True),      # five strips, the last one half
    (20, 80, 82, 64, 128, 0, (8, 8), 0.5, False, True, True),    # eight strips
    (9, 97, 83, 72, 104, 1, (8, 8), 0.25, True, True, True),
    (12, 64, 100, 96, 104, 1, (8, 8), 0.25, True, False, True),  # seven
    (1, 149, 131, 56, 64, 1, (8, 8), 0.75, False, True, False),
    (9, 47, 53, 64, 64, 1, (8, 8), 0.5, True, True, True),
    (16, 73, 73, 80, 192, 0, (8, 8), 0.5, True, True, True),     # twelve strips
    (28, 29, 27, 32, 256, 1, (8, 8), 0.5, False, True, False),   # sixteen
    # patches smaller than the spill area and the biases, several tiles a workgroup
    (8, 56, 56, 8, 256, 1, (8, 8), 1.0, False, True, False),
    (16, 56, 56, 8, 184, 1, (8, 8), 1.0, True, False, False),
    (8, 56, 56, 8, 256, 0, (4, 16), 1.0, False, False, False),   # no bias
    (64, 16, 16, 8, 256, 1, (8, 8), 1.0, False, False, True),
    (12, 64, 100, 72, 104, 1, (8, 8), 0.25, False, False, True),
    (19, 60, 61, 56, 40, 1, (8, 8), 0.25, False, False, False),  # three strips of few steps: a strip that drops the last unit
]


@pytest.mark.parametrize("n", range(len(CASES)))
def test_bands(n):
    import torch
    B, L, J, I, O, pad, (bo, bi), density, residual, relu, band = CASES[n]
    print("bands case", n, CASES[n], flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    gamma = (np.random.default_rng(n).random((-(-O // bo), -(-I // bi))) < density).astype(np.uint8)
    gamma[0, 0] = 1
    gamma[1] = 0                     # a block row with nothing
    W = (torch.randn(O, 3, 3, I, generator=gen, device="cuda") * (2.0 / (9 * I * density)) ** 0.5).bfloat16()
    bias = np.random.default_rng(n).standard_normal(O).astype(np.float32) if n % 4 else None
    layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, bo, bi, "bf16", bias=bias)
    X = torch.randn(B, L, J, I, generator=gen, device="cuda").bfloat16()
    shape = layer.out_shape(B, L, J, (1, 1), (pad, pad))
    R = torch.randn(shape, generator=gen, device="cuda").bfloat16() if residual else None

    def run(x, kernel):
        out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        ran = kernels_of(lambda: layer.conv2d(x, (1, 1), (pad, pad), out=out, residual=R, relu=relu))
        assert any(kernel in k for k in ran), ran
        return out

    rows = layer.plan[layer.plan[24]:]   # the plan's row-band section
    steps = int(rows[11])
    depth = 3 if steps <= 3 else 5 if steps <= 5 else 6
    out = run(X, "conv_bands<%d, %d, %s>" % (depth, 1024 if depth == 3 else 768, str(residual).lower()))
    Xinf = X.clone()
    Xinf[B - 1, 0, 2] = float("inf")
    Xinf[B // 2, L // 2, 4, I - 1] = float("nan")
    oinf = run(Xinf, "conv_bands<")
    far = torch.ones(shape[:3], dtype=torch.bool, device="cuda")   # what no window with one of these reaches
    for b, y, x in ((B - 1, 0, 2), (B // 2, L // 2, 4)):
        far[b, max(0, y - 2 + pad):y + 1 + pad, max(0, x - 2 + pad):x + 1 + pad] = False
    assert bool((oinf.view(torch.int16) == out.view(torch.int16))[far].all())
    if not relu:                         # (an activation hides them)
        # a strip's rows share what one of them keeps: what keeps the last unit has the NaN, strips without it do not
        keeps = torch.from_numpy(np.repeat(gamma[:, (I - 1) // bi], bo)[:O].astype(bool)).cuda()
        strip = rows[rows[5]:rows[5] + 4 * rows[0]].reshape(-1, 4)
        shares = torch.zeros(O, dtype=torch.bool, device="cuda")
        for first in strip.tolist():
            chans = [c + k for c in first if c >= 0 for k in range(4)]
            shares[chans] = bool(keeps[chans].any())
        hit = ~far
        hit[B - 1] &= B - 1 == B // 2    # (the other image's pixel is infinite in every channel)
        assert bool(oinf[hit][:, keeps].isnan().all()) and bool(torch.isfinite(oinf[hit][:, ~shares]).all())
        everything = torch.from_numpy(np.repeat(gamma.any(1), bo)[:O].copy()).cuda()
        assert not bool(torch.isfinite(oinf[B - 1][~far[B - 1]][:, everything]).any())
    if band:
        layer.struct.kernels = bsp.BSP_KERNEL_BAND
        assert bool((out.view(torch.int16) == run(X, "conv_band3<").view(torch.int16)).all())
        want = run(Xinf, "conv_band3<")
        same = (oinf.view(torch.int16) == want.view(torch.int16)) | (oinf.isnan() & want.isnan())
        assert bool(same.all())
        return
    keep = torch.from_numpy(np.kron(gamma, np.ones((bo, bi), np.uint8))[:O, :I].copy()).cuda()
    want = conv_fp64(X, W * keep[:, None, None, :], 1, (pad, pad))
    if bias is not None:
        want += torch.from_numpy(bias).cuda()
    if residual:  # the stored result takes the residual: a second rounding
        want = want.bfloat16().double() + R.double()
    if relu:
        want = want.clamp_min(0)
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    # one rounding to bf16 is 3.9e-3 at most, the fused epilogue has two and may round a sum the other way in the first
    assert bool(((out.double() - want).abs() <= (1.2e-2 if residual else 6e-3) * scale).all())


@pytest.mark.parametrize("B", [1, 3, 7, 8, 9, 13, 16])
def test_band_kernel_with_images_left_over(B):
    """Batches that are and are no multiple of eight, which take an instance each: every band is computed by some XCD."""
    import torch
    print("band kernel, batch", B, flush=True)
    gen = torch.Generator("cuda").manual_seed(B)
    gamma = (np.random.default_rng(B).random((16, 9)) < 0.5).astype(np.uint8)
    W = (torch.randn(128, 3, 3, 72, generator=gen, device="cuda") * 0.05).bfloat16()
    layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, 8, 8, "bf16")
    layer.struct.kernels = bsp.BSP_KERNEL_BAND
    X = torch.randn(B, 37, 53, 72, generator=gen, device="cuda").bfloat16()
    out = torch.full(layer.out_shape(B, 37, 53, (1, 1), (1, 1)), float("nan"), dtype=torch.bfloat16, device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (1, 1), (1, 1), out=out))
    assert any("conv_band3<" in k for k in ran), ran
    keep = torch.from_numpy(np.kron(gamma, np.ones((8, 8), np.uint8))).cuda()
    want = conv_fp64(X, W * keep[:, None, None, :], 1, (1, 1))
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 6e-3 * scale).all())
