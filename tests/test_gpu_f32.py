"""Single-precision layers through the dispatcher against the oracle at the sizes where the
kernels' tiles, chunks and slabs end (needs a GPU)."""
import numpy as np
import pytest

import oracle
import paper_2407_09453_amd as bsp
from synthetic import draw_layer

from gpu_util import TOL, conv_fp64, kernels_of, make_layer, to_device, to_host

pytestmark = pytest.mark.gpu

# B, L, J, I, O, H, K, stride, pad
SHAPES = [
    (1, 1, 1, 8, 8, 1, 1, 1, 0),            # one pixel, one block
    (1, 1, 63, 40, 20, 1, 1, 1, 0),         # last lanes of a pixel tile idle; more waves than blocks
    (65, 1, 1, 130, 12, 1, 1, 1, 0),        # two pixel tiles, channels that are not whole pieces
    (256, 1, 1, 520, 72, 1, 1, 1, 0),       # the most pixels read without staging
    (257, 1, 1, 520, 72, 1, 1, 1, 0),       # the fewest staged
    (2, 9, 64, 24, 40, 3, 3, 1, 1),         # rows of exactly one chunk
    (1, 5, 65, 17, 9, 3, 3, 1, 1),          # rows of two chunks, ragged channels
    (1, 31, 129, 48, 64, 3, 3, 2, 1),       # three chunks, strided
    (2, 13, 11, 70, 136, 5, 5, 1, 2),       # several slabs, ragged last block column
    (1, 20, 20, 33, 24, 1, 7, 2, 3),        # one-row window, strided: rows in between are not staged
    (1, 20, 20, 33, 24, 7, 1, 2, 3),
    (3, 30, 30, 64, 64, 1, 1, 2, 0),        # strided pointwise
    (1, 7, 7, 512, 64, 3, 3, 1, 1),         # few pixels, long contraction: block rows shared by waves
    (4, 56, 56, 64, 64, 3, 3, 1, 1),        # many tiles per workgroup row
    (1, 6, 7, 16, 16, 3, 3, 1, 4),          # padding wider than the window
]


def _assert_close(y, ref, terms, what):
    """Every element within the stated 1e-5, and the whole result within the 2-norm that a sum
    of `terms` products in fp32 can show: n additions, each rounding by at most 2^-24 of a partial
    sum that grows like sqrt(k), add up to about sqrt(n / 6) * 2^-24; allowed is twice that."""
    rms = float(np.sqrt(np.mean(ref * ref)))
    err = np.abs(y - ref)
    assert np.isfinite(y).all(), what
    assert (err <= TOL["f32"] * np.maximum(np.abs(ref), rms)).all(), what
    rel = float(np.sqrt(np.mean(err * err))) / max(rms, 1e-30)
    assert rel <= 2 * np.sqrt(max(terms, 24) / 6) * 2.0 ** -24, (what, rel)


OFF_X3 = 26  # the plan's header word that says where its three-part section is (csrc/bsp_plan.h)


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("fused", [False, True], ids=["plain", "fused"])
@pytest.mark.parametrize("parts", [True, False], ids=["as packed", "without parts"])
def test_f32_shapes(bo, bi, fused, parts):
    """As the dispatcher sends them, and the whole chunks of channels among them with a plan that has no three-part
    section, as plans of layers past its limits: on the kernels before that one."""
    import torch
    for n, (B, L, J, I, O, H, K, s, p) in enumerate(SHAPES):
        if I % 8 and not parts:
            continue
        pad = (p if H > 1 or K == 1 else 0, p if K > 1 or H == 1 else 0)
        c = draw_layer("t", B=B, L=L, J=J, I=I, O=O, H=H, K=K, stride=(s, s), pad=pad, bo=bo, bi=bi, dtype="f32",
                       mask_kind="bernoulli", density=0.5, seed=9100 + n, b_std=0.5)
        print("case", n, SHAPES[n], bo, bi, fused, flush=True)
        layer = make_layer(c)
        if not parts:
            layer.plan[OFF_X3] = 0
            assert not any("conv_f32x3" in k for k in kernels_of(lambda: layer.conv2d(to_device(c), c.stride, c.pad)))
        Y = torch.full((c.B, c.M, c.N, c.O), float("nan"), device="cuda")
        if fused:
            r = np.random.default_rng(n).standard_normal(tuple(Y.shape)).astype(np.float32)
            layer.conv2d(to_device(c), c.stride, c.pad, out=Y, residual=torch.from_numpy(r).cuda(), relu=True)
            ref = oracle.conv2d_fused(c.X, c.W, c.bias, c.gamma, bo, bi, c.stride, c.pad, residual=r, relu=True, dtype="f32")
        else:
            layer.conv2d(to_device(c), c.stride, c.pad, out=Y)
            ref = oracle.conv2d(c.X, c.W, c.bias, c.gamma, bo, bi, c.stride, c.pad)
        torch.cuda.synchronize()
        _assert_close(to_host(Y), ref, I * H * K, f"shape {n}")


def _check_on_gpu(kernel, gran, B, L, J, I, O, H, K, s, density):
    """One layer against fp64, its kept blocks drawn block row by block row with the given densities in
    turn; `kernel` is what has to run it."""
    import torch
    bo, bi = gran
    gen = torch.Generator("cuda").manual_seed(I + O)
    rng = np.random.default_rng(I + O)
    nbr, nbc = -(-O // bo), -(-I // bi)
    gamma = (rng.random((nbr, nbc)) < np.resize(density, nbr)[:, None]).astype(np.uint8)
    keep = torch.from_numpy(np.kron(gamma, np.ones(gran, np.uint8))[:O, :I].copy()).cuda()[:, None, None, :]
    X = torch.randn(B, L, J, I, generator=gen, device="cuda")
    W = torch.randn(O, H, K, I, generator=gen, device="cuda")
    R = torch.randn((B, (L - 1) // s + 1, (J - 1) // s + 1, O), generator=gen, device="cuda")
    bias = rng.standard_normal(O).astype(np.float32)
    layer = bsp.BspLayer(W.cpu().numpy(), gamma, bo, bi, "f32", bias=bias)
    ref = conv_fp64(X, W * keep, s, (H // 2, K // 2)) + torch.from_numpy(bias).cuda()
    rms = ref.pow(2).mean().sqrt()
    terms = max(float(max(density)) * I * H * K, 24)
    sigma = (terms / 6) ** 0.5 * 2.0 ** -24     # of a sum of so many terms, as above
    for fused in (False, True):
        Y = torch.full(tuple(R.shape), float("nan"), device="cuda")
        args = dict(residual=R, relu=True) if fused else {}
        ran = kernels_of(lambda: layer.conv2d(X, (s, s), (H // 2, K // 2), out=Y, **args))
        assert any(kernel in k for k in ran), ran
        want = (ref + R).clamp_min(0) if fused else ref
        err = (Y - want).abs()
        assert bool((err <= max(TOL["f32"], 8 * sigma) * torch.maximum(ref.abs(), rms)).all()), (gran, fused)
        assert float(err.pow(2).mean().sqrt() / rms) <= 2 * sigma, (gran, fused)


GRANS = [(8, 8), (4, 16), (16, 4)]
UNEVEN = (1.0, 0.83, 0.0, 0.6, 0.97)


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("shape", [(16, 28, 28, 61, 1, 1, 1), (8, 57, 57, 109, 1, 1, 2), (12, 57, 57, 109, 1, 3, 1)])
def test_rows_of_more_than_64_blocks(gran, shape):
    """Many pixels, so that no two waves share a row of up to 138 blocks: a wave asks for the row's next 64
    columns in the middle of a slab, at another place in every row; one row is empty."""
    B, L, J, O, H, K, s = shape
    _check_on_gpu("conv_f32<%d, %d" % gran, gran, B, L, J, gran[1] * 138 - 3, O, H, K, s, UNEVEN)


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("shape", [(63, 55, 57, 93, 205, 1, 1, 1), (63, 55, 57, 93, 204, 1, 1, 2), (32, 56, 57, 29, 205, 3, 3, 1)])
def test_widest_pixel_tiles(gran, shape):
    """Four lane tiles a wave (two with 16x4 blocks), ragged channels and pixels that do not fill the last tile."""
    tiles = 2 if gran[0] == 16 else 4
    _check_on_gpu("conv_f32<%d, %d, %d>" % (*gran, tiles), gran, *shape, (1.0, 0.9, 0.7))


@pytest.mark.parametrize("gran", GRANS)
@pytest.mark.parametrize("rows", [1, 65])
def test_fc_rows_of_more_than_64_blocks_a_wave(gran, rows):
    """Long rows without staging: sixteen waves share them, 128 blocks each and a few more."""
    _check_on_gpu("fc_f32<%d, %d>" % gran, gran, rows, 1, 1, gran[1] * (16 * 128 + 3) - 1, 37, 1, 1, 1, (1.0, 0.96, 0.0))
