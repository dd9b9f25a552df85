"""Single-precision layers on the three-part kernel (csrc/bsp_f32x3.hip), through the dispatcher: against fp64,
and with values that three bf16 parts cannot hold (needs a GPU)."""
import numpy as np
import pytest

import paper_2407_09453_amd as bsp

from gpu_util import conv_fp64, kernels_of

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, L, J, I, O, H, K, stride, blocks, density
    (2, 9, 11, 16, 24, 3, 3, 1, (8, 8), 0.5),        # one slab, two strips, ragged tiles
    (1, 30, 30, 136, 50, 1, 1, 1, (8, 8), 0.5),      # results one by one
    (4, 17, 17, 64, 64, 1, 7, 1, (8, 8), 0.5),
    (2, 13, 10, 72, 40, 5, 5, 2, (16, 4), 0.5),      # two slabs, the second of one chunk
    (2, 20, 21, 264, 56, 3, 1, 2, (16, 4), 0.75),    # five slabs, one row of the window at a stride
    (8, 56, 56, 256, 64, 1, 1, 1, (8, 8), 0.25),     # a plain matrix product
    (3, 29, 41, 1032, 72, 1, 1, 2, (16, 4), 0.5),    # slabs of 256 channels
    (4, 35, 35, 96, 100, 3, 3, 1, (4, 16), 0.5),     # four block rows a strip
    (2, 14, 14, 256, 256, 3, 3, 1, (8, 8), 1.0),     # waves share a strip's steps
    (300, 7, 5, 24, 136, 2, 2, 1, (8, 8), 0.5),
]


def _layer(n, scale=1.0):
    import torch
    B, L, J, I, O, H, K, s, (bo, bi), density = SHAPES[n]
    gen = torch.Generator("cuda").manual_seed(n)
    rng = np.random.default_rng(n)
    gamma = (rng.random((-(-O // bo), -(-I // bi))) < density).astype(np.uint8)
    gamma[1] = 0
    gamma[0, 0] = 1
    keep = torch.from_numpy(np.kron(gamma, np.ones((bo, bi), np.uint8))[:O, :I].copy()).cuda()[:, None, None, :]
    X = torch.randn(B, L, J, I, generator=gen, device="cuda")
    W = torch.randn(O, H, K, I, generator=gen, device="cuda") * scale
    bias = rng.standard_normal(O).astype(np.float32)
    return X, W, keep, gamma, bias, bsp.BspLayer(W.cpu().numpy(), gamma, bo, bi, "f32", bias=bias), (H // 2, K // 2)


@pytest.mark.parametrize("n", range(len(SHAPES)))
def test_against_fp64(n):
    import torch
    X, W, keep, gamma, bias, layer, pad = _layer(n)
    B, L, J, I, O, H, K, s, (bo, bi), density = SHAPES[n]
    print("three-part case", n, SHAPES[n], flush=True)
    out = torch.full(layer.out_shape(B, L, J, (s, s), pad), float("nan"), device="cuda")
    ran = kernels_of(lambda: layer.conv2d(X, (s, s), pad, out=out))
    assert any("conv_f32x3" in k for k in ran), ran
    want = conv_fp64(X, W * keep, s, pad) + torch.from_numpy(bias).cuda()
    rms = want.pow(2).mean().sqrt()
    # a sum of n products takes n / 32 roundings of 2^-24 at most for the leading parts and the others are
    # 2^-8 of them; four standard deviations of a multiply-add chain's would be eight times this
    sigma = (max(density * I * H * K, 24) / 6) ** 0.5 * 2.0 ** -24
    err = (out.double() - want).abs()
    assert float(err.pow(2).mean().sqrt() / rms) <= sigma
    assert bool((err <= max(1e-5, 8 * sigma) * torch.maximum(want.abs(), rms)).all())
    R = torch.randn(out.shape, generator=torch.Generator("cuda").manual_seed(99), device="cuda")
    assert torch.equal(layer.conv2d(X, (s, s), pad, residual=R, relu=True), torch.relu(out + R))


@pytest.mark.parametrize("n", [0, 3, 7, 8])
@pytest.mark.parametrize("what", ["tiny", "huge", "inf", "nan"])
def test_values_beyond_three_parts(n, what):
    """Results are those of an fp32 sum over kept blocks: a dropped channel's infinity reaches nothing, values
    below 2^-100 keep their bits, values near the largest are no infinities."""
    import torch
    X, W, keep, gamma, bias, layer, pad = _layer(n, 2.0 ** -20 if what == "huge" else 1.0)
    B, L, J, I, O, H, K, s, (bo, bi), density = SHAPES[n]
    c = int(np.argmin(gamma.sum(0)))  # a block column that some block rows drop
    assert gamma[1].sum() == 0
    if what == "tiny":
        X[0] *= 2.0 ** -115
    elif what == "huge":
        X[0, 3, 3, c * bi] = 3.4e38
    else:
        X[0, 3, 3, c * bi] = float(what)
        X[B - 1, 2, 4, 0] = -float(what)
    got = layer.conv2d(X, (s, s), pad).double()
    # the reference sums a block row's kept channels only: where a channel is dropped its value is zero
    rows = torch.from_numpy(np.repeat(gamma, bo, 0)[:O].astype(bool)).cuda()
    want = torch.empty_like(got)
    for r in range(gamma.shape[0]):
        o = slice(r * bo, min(O, (r + 1) * bo))
        kept = torch.from_numpy(np.repeat(gamma[r], bi)[:I].astype(bool)).cuda()
        want[..., o] = conv_fp64(torch.where(kept, X, 0.0), W[o] * keep[o], s, pad) if kept.any() else 0.0
    want += torch.from_numpy(bias).cuda()
    finite = want.isfinite() & (want.abs() < 3.4e38)
    assert torch.equal(got.isfinite(), finite)
    assert torch.equal(got.isnan(), want.isnan())
    if what == "tiny":  # (without the bias, which hides them)
        bare = bsp.BspLayer(W.cpu().numpy(), gamma, bo, bi, "f32")
        got, want = bare.conv2d(X, (s, s), pad)[0].double(), (want - torch.from_numpy(bias).cuda())[0]
        want = conv_fp64(X[:1], W * keep, s, pad)[0]
        finite = torch.ones_like(want, dtype=torch.bool)
    err, ref = (got - want).abs()[finite], want[finite]
    assert bool((err <= 1e-5 * torch.maximum(ref.abs(), ref[ref.abs() < 1e30].pow(2).mean().sqrt())).all())


def test_weights_beyond_three_parts_stay_on_the_fp32_kernel():
    X, W, keep, gamma, bias, layer, pad = _layer(2)
    W = W.cpu().numpy()
    W[0, 0, 0, 0] = 1e-35
    ran = kernels_of(lambda: bsp.BspLayer(W, gamma, 8, 8, "f32", bias=bias).conv2d(X, (1, 1), pad))
    assert any("conv_f32<" in k for k in ran), ran


@pytest.mark.parametrize("I", [64, 128, 136])
def test_sums_of_one_product(I):
    """One-hot inputs.  Up to sixteen chunks eight of the nine products of parts are summed: what is left out is
    2^-34 of the product, and the minor ones' sum, at most 2^-6 of it, is rounded twice after the small ones, together
    less than 2^-7 of a unit in the last place.  Beyond them six: 2^-24 of the product is left out at the most."""
    import torch
    gen = torch.Generator("cuda").manual_seed(7)
    B, L, O = 8, 40, 64
    W = torch.randn(O, 1, 1, I, generator=gen, device="cuda")
    x = torch.randn(B, L, L, generator=gen, device="cuda")
    x[0, 0] = W[:, 0, 0, 0] = 1 + 2.0 ** -8 - 2.0 ** -17  # the parts with the largest minor products
    at = torch.randint(0, I, (B, L, L, 1), generator=gen, device="cuda")
    at[0, 0] = 0
    X = torch.zeros(B, L, L, I, device="cuda").scatter_(3, at, x[..., None])
    layer = bsp.BspLayer(W.cpu().numpy(), np.ones((8, I // 8), np.uint8), 8, 8, "f32")
    ran = kernels_of(lambda: layer.conv2d(X))
    assert any("conv_f32x3" in k for k in ran), ran
    want = x.double()[..., None] * W.view(O, I).t()[at[..., 0]].double()
    ulp = torch.pow(2.0, torch.floor(torch.log2(want.abs())) - 23)
    out = 0.0 if I <= 128 else 2.0 ** -24 * want.abs()
    assert bool(((layer.conv2d(X).double() - want).abs() <= out + (0.5 + 2.0 ** -7) * ulp).all())
