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
    (2, 10, 10, 512, 64, 3, 3, 1, (16, 4), 0.75),    # four lane tiles: four waves share a strip's steps
    (6, 40, 40, 64, 40, 3, 3, 1, (4, 16), 0.5),      # two of them; five output block rows in a strip and a half
    (16, 40, 40, 64, 64, 3, 3, 1, (8, 8), 0.5),      # two groups of pixels
    (8, 28, 28, 128, 512, 1, 1, 1, (8, 8), 0.5),     # a plain matrix product of few steps
    (1, 23, 19, 1032, 1034, 1, 1, 1, (8, 8), 0.5),   # weights from the payload, a strip that is not full
    (2, 25, 27, 2048, 520, 1, 1, 2, (16, 4), 0.5),
    (4, 30, 31, 1024, 1040, 1, 1, 1, (4, 16), 0.25),
    (8, 31, 28, 1032, 1034, 1, 1, 1, (16, 4), 0.1),
    (1, 23, 19, 1032, 1032, 1, 1, 1, (8, 8), 0.03),  # few steps
    (8, 30, 30, 1032, 1032, 1, 1, 1, (8, 8), 0.03),
]
TILES = [2, 2, 2, 2, 2, 2, 2, 2, 2, 4, 4, 4, 4, 4, 2, 2, 2, 4, 2, 4]  # lane tiles of a wave


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
    assert any("conv_f32x3<%d" % TILES[n] in k for k in ran), ran
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


@pytest.mark.parametrize("n", [0, 3, 5, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19])
@pytest.mark.parametrize("what", ["huge", "sums", "inf", "nan"])
def test_values_beyond_three_parts(n, what):
    """Results are those of an fp32 sum over kept blocks: a dropped channel's infinity reaches nothing, values
    and sums near the largest are no infinities."""
    import torch
    X, W, keep, gamma, bias, layer, pad = _layer(n, {"huge": 2.0 ** -20, "sums": 2.0 ** 15}.get(what, 1.0))
    B, L, J, I, O, H, K, s, (bo, bi), density = SHAPES[n]
    print("beyond three parts", n, SHAPES[n], what, flush=True)
    c = int(np.argmin(gamma.sum(0)))  # a block column that some block rows drop
    assert gamma[1].sum() == 0
    if what == "huge":
        X[0, 3, 3, c * bi] = 3.4e38
    elif what == "sums":
        X[0] *= 2.0 ** 100
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
    if what == "sums":  # (the first image's sums are of another size than the others')
        got, want, finite = got[0], want[0], finite[0]
    err, ref = (got - want).abs()[finite], want[finite]
    rms = ref[ref.abs() < (1e37 if what == "sums" else 1e30)].pow(2).mean().sqrt()
    assert bool((err <= 1e-5 * torch.maximum(ref.abs(), rms)).all())


def _three_parts(x):
    """x as far as three bf16 parts hold it."""
    parts, rest = 0.0, x.cpu()
    for _ in range(3):
        part = rest.bfloat16().float()
        parts, rest = parts + part.double(), rest - part
    return parts.cuda()


@pytest.mark.parametrize("n", [0, 3, 5, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 17, 18, 19])
@pytest.mark.parametrize("rows", ["all", "half"])
def test_small_values_keep_their_bits(n, rows):
    """Values near the smallest float, of which three bf16 parts hold ten bits unless they are scaled: the results that
    they alone make keep the accuracy of an fp32 sum, beside others in the same tile that no bit of theirs reaches."""
    import torch
    X, W, keep, gamma, bias, layer, pad = _layer(n)
    B, L, J, I, O, H, K, s, (bo, bi), density = SHAPES[n]
    print("small values", n, SHAPES[n], rows, flush=True)
    top = L if rows == "all" else L // 2
    X[0, :top] *= 2.0 ** -125
    X[0, 0] = 0.0
    bare = bsp.BspLayer(W.cpu().numpy(), gamma, bo, bi, "f32")  # (a bias would hide them)
    got, want = bare.conv2d(X, (s, s), pad)[0].double(), conv_fp64(X[:1], W * keep, s, pad)[0]
    parts = conv_fp64(_three_parts(X[:1]), W * keep, s, pad)[0]
    last = (top - 1 + pad[0] - (H - 1)) // s if rows == "half" else want.shape[0] - 1  # output rows of small values alone
    sigma = (max(density * I * H * K, 24) / 6) ** 0.5 * 2.0 ** -24  # as above
    bound = max(1e-6, 16 * sigma)
    for a, b, alone in ((0, last + 1, True), (last + H, want.shape[0], False)):
        if a >= b:
            continue
        g, v = got[a:b], want[a:b]
        scale = torch.maximum(v.abs(), v.pow(2).mean().sqrt())
        assert bool(((g - v).abs() <= bound * scale).all()), (a, b)
        if alone:  # (the bound sees what the parts of unscaled values lose)
            assert bool(((parts[a:b] - v).abs() > 4 * bound * scale).any())


@pytest.mark.parametrize("x,w", [(-55, -55), (-62, -62), (-90, -36), (-130, 0), (-64, -66)])
def test_small_products_keep_their_bits(x, w):
    """Products down to the smallest floats, one to a sum: within what test_sums_of_one_product allows, and, where the
    result has fewer than 24 bits, the rounding to those (a quarter of a place at the most) and then to its own."""
    import torch
    gen = torch.Generator("cuda").manual_seed(x * 1000 + w)
    B, L, I, O = 8, 40, 64, 64
    W = torch.randn(O, 1, 1, I, generator=gen, device="cuda") * 2.0 ** w
    v = torch.randn(B, L, L, generator=gen, device="cuda") * 2.0 ** x
    at = torch.randint(0, I, (B, L, L, 1), generator=gen, device="cuda")
    X = torch.zeros(B, L, L, I, device="cuda").scatter_(3, at, v[..., None])
    layer = bsp.BspLayer(W.cpu().numpy(), np.ones((8, 8), np.uint8), 8, 8, "f32")
    ran = kernels_of(lambda: layer.conv2d(X))
    assert any("conv_f32x3" in k for k in ran), ran
    want = v.double()[..., None] * W.view(O, I).t()[at[..., 0]].double()
    place = torch.pow(2.0, torch.floor(torch.log2(want.abs())).clamp_min(-126) - 23)
    most = 0.5 + 2.0 ** -7 + 0.25 * (want.abs() < 2.0 ** -126)
    assert bool(((layer.conv2d(X).double() - want).abs() <= most * place).all())


def _fastest(call, n=20):
    import torch
    call()
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(n):
            call()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) / n)
    return best


def test_rare_values_cost_little():
    """One activation near the smallest float, one in a hundred, or all of them: within 1.5 times the time without any
    (6, 18 and 18 times while the tiles that held one were summed a second time).  One NaN: twice (3.3 times while
    its tile was summed with one product in flight)."""
    import torch
    gen = torch.Generator("cuda").manual_seed(3)
    gamma = (np.random.default_rng(3).random((8, 8)) < 0.5).astype(np.uint8)
    layer = bsp.BspLayer(torch.randn(64, 3, 3, 64, generator=gen, device="cuda").cpu().numpy(), gamma, 8, 8, "f32")
    X = torch.randn(32, 56, 56, 64, generator=gen, device="cuda")
    out = torch.empty(32, 56, 56, 64, device="cuda")
    timed = lambda x: _fastest(lambda: layer.conv2d(x, (1, 1), (1, 1), out=out))
    base = timed(X)
    one, many, nan = X.clone(), X.clone(), X.clone()
    one[0, 3, 3, 5] = 1e-36
    many[torch.rand(X.shape, generator=gen, device="cuda") < 0.01] = 1e-36
    nan[0, 3, 3, 5] = float("nan")
    times = [timed(x) / base for x in (one, many, X * 1e-36, nan)]
    print("times of the time without such values:", times, flush=True)
    assert max(times[:3]) <= 1.5 and times[3] <= 2, times


@pytest.mark.parametrize("value", [1e-35, 3e38, float("inf"), float("nan")])
def test_weights_beyond_three_parts_stay_on_the_fp32_kernel(value):
    """A layer with such a weight in a kept block, and what becomes of its results."""
    import torch
    n = 2
    X, W, keep, gamma, bias, _, pad = _layer(n)
    X *= 0.25  # (the largest weight's products stay below the largest float)
    W[0, 0, 0, 0] = value
    layer = bsp.BspLayer(W.cpu().numpy(), gamma, 8, 8, "f32", bias=bias)
    got = layer.conv2d(X, (1, 1), pad).double()
    ran = kernels_of(lambda: layer.conv2d(X, (1, 1), pad))
    assert any("conv_f32<" in k for k in ran), ran
    assert keep[0, 0, 0, 0] == 1
    want = conv_fp64(X, torch.where(keep.bool(), W, 0.0), 1, pad) + torch.from_numpy(bias).cuda()
    assert torch.equal(got.isnan(), want.isnan())
    finite = want.isfinite() & (want.abs() < 3.4e38)
    assert torch.equal(got.isfinite(), finite)
    err, ref = (got - want).abs()[finite], want[finite]
    assert bool((err <= 1e-5 * torch.maximum(ref.abs(), ref[ref.abs() < 1e30].pow(2).mean().sqrt())).all())


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
