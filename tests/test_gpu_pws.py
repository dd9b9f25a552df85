"""The kernel that streams pixels past weights in registers (csrc/bsp_pws.hip) through the dispatcher, bit for bit
against the pointwise kernel, whose steps it takes: every length of strip, pixels and strips that fill no tile or
workgroup, strides, infinities, biases near the ends of 32 bits (needs a GPU)."""
import numpy as np
import pytest

import paper_2407_09453_amd as bsp

from gpu_util import conv_fp64, kernels_of

pytestmark = pytest.mark.gpu

BF16 = [
    # B, L, J, I, O, stride, blocks, density, residual, relu
    (33, 33, 31, 64, 128, 1, (8, 8), 1.0, True, True),       # two steps, eight strips, a last tile of 31 pixels
    (19, 61, 63, 64, 256, 1, (8, 8), 0.5, False, True),      # sixteen strips, two workgroups a pixel
    (7, 131, 41, 24, 72, 1, (8, 8), 0.75, True, False),      # one step, five strips, an odd number of pieces a pixel
    (5, 101, 77, 72, 280, 1, (4, 16), 0.5, True, True),      # strips of four block rows; 18 of them, four at a time
    (6, 141, 139, 112, 232, 2, (8, 8), 0.5, False, False),   # every second pixel
    (34, 32, 32, 128, 128, 1, (16, 4), 0.5, True, True),     # half pieces
    (3, 113, 111, 192, 104, 1, (8, 8), 1.0, False, True),    # six steps, two loads a lane
    (3, 113, 111, 192, 104, 1, (16, 4), 1.0, True, False),
    (2, 150, 149, 256, 192, 1, (8, 8), 1.0, True, True),     # eight steps
    (9, 95, 93, 512, 64, 1, (16, 4), 0.25, False, False),    # four loads a lane
    (3, 120, 118, 440, 120, 1, (8, 8), 0.25, True, True),
    (2, 99, 97, 384, 128, 1, (8, 8), 1.0, True, True),       # twelve steps: tiles of 16 pixels
    (2, 99, 97, 360, 256, 1, (4, 16), 1.0, False, True),     # sixteen waves
    (3, 89, 87, 512, 128, 1, (16, 4), 1.0, False, True),     # sixteen steps
    (2, 101, 99, 504, 264, 1, (8, 8), 1.0, True, False),
    (17, 64, 64, 256, 32, 1, (8, 8), 0.75, False, False),     # two strips on eight waves
    (2, 101, 99, 1024, 256, 1, (16, 4), 0.4, True, True),    # units to 255, sixteen waves with two loads a lane
    (2, 101, 99, 1024, 256, 1, (16, 4), 0.4, False, False),
]


def _same(layer, call, shape, dtype, bits):
    import torch
    fill = float("nan") if dtype == torch.bfloat16 else 77
    out = torch.full(shape, fill, dtype=dtype, device="cuda")
    ran = kernels_of(lambda: call(out))
    assert any("conv_pws<" in k for k in ran), ran
    want = torch.full(shape, fill, dtype=dtype, device="cuda")
    layer.struct.kernels = bsp.BSP_KERNEL_PW
    ran = kernels_of(lambda: call(want))
    assert any("conv_pw<" in k for k in ran), ran
    assert bool((out.view(bits) == want.view(bits)).all())
    return out


def _mask(n, O, I, bo, bi, density):
    gamma = (np.random.default_rng(n).random((-(-O // bo), -(-I // bi))) < density).astype(np.uint8)
    gamma[0, 0] = 1
    gamma[1] = 0                     # a block row with nothing
    return gamma


@pytest.mark.parametrize("n", range(len(BF16)))
def test_bf16(n):
    import torch
    B, L, J, I, O, s, (bo, bi), density, residual, relu = BF16[n]
    print("pws case", n, BF16[n], flush=True)
    gen = torch.Generator("cuda").manual_seed(n)
    gamma = _mask(n, O, I, bo, bi, density)
    W = torch.randn(O, 1, 1, I, generator=gen, device="cuda").bfloat16().float().cpu().numpy()
    layer = bsp.BspLayer(W, gamma, bo, bi, "bf16", bias=np.random.default_rng(n).standard_normal(O).astype(np.float32) if n % 4 else None)
    X = torch.randn(B, L, J, I, generator=gen, device="cuda").bfloat16()
    X[B - 1, 0, 2] = float("inf")    # reach what keeps their channels, and no other pixel
    X[B // 2, L // 2, 4, I - 1] = float("nan")
    shape = layer.out_shape(B, L, J, (s, s), (0, 0))
    R = torch.randn(shape, generator=gen, device="cuda").bfloat16() if residual else None
    out = _same(layer, lambda y: layer.conv2d(X, (s, s), (0, 0), out=y, residual=R, relu=relu), shape, torch.bfloat16, torch.int16)
    assert int((~torch.isfinite(out)).any(-1).sum()) <= 2


I8 = [
    # B, L, J, I, O, blocks, density, shift, the largest bias
    (9, 61, 63, 64, 256, (8, 8), 1.0, 8, 5000),          # one step: two strips a wave
    (9, 61, 63, 48, 208, (4, 16), 0.5, 0, 50),           # no rounding
    (49, 33, 31, 64, 112, (16, 4), 0.75, 9, 5000),       # seven strips
    (9, 61, 63, 128, 256, (8, 8), 0.5, 10, 5000),        # two steps
    (34, 32, 32, 256, 128, (8, 8), 1.0, 11, 5000),       # four
    (3, 113, 111, 384, 112, (16, 4), 1.0, 11, 5000),     # six
    (4, 95, 93, 512, 128, (8, 8), 1.0, 12, 5000),        # eight
    (4, 95, 93, 1008, 128, (8, 8), 0.1, 12, 5000),       # four loads a lane
    (9, 61, 63, 64, 256, (8, 8), 1.0, 22, 2**30),        # the last biases and shift on the short way to rescale,
    (9, 61, 63, 64, 256, (8, 8), 1.0, 22, 2**30 + 40),   # the first on the long one
    (9, 61, 63, 128, 256, (8, 8), 1.0, 23, 2**30),
    (9, 61, 63, 128, 256, (8, 8), 1.0, 31, 2**31 - 1),
    (34, 32, 32, 256, 128, (8, 8), 1.0, 1, 2**31 - 1),
]


@pytest.mark.parametrize("n", range(len(I8)))
def test_i8(n):
    import torch
    B, L, J, I, O, (bo, bi), density, shift, most = I8[n]
    print("pws int8 case", n, I8[n], flush=True)
    rng = np.random.default_rng(n)
    W = rng.integers(-127, 128, (O, 1, 1, I), dtype=np.int8)
    bias = rng.integers(-most, most + 1, O).astype(np.int32)
    bias[::7], bias[3::7] = most, -most
    layer = bsp.BspLayerI8(W, _mask(n, O, I, bo, bi, density), bo, bi, bias=bias)
    X = torch.from_numpy(rng.integers(-128, 128, (B, L, J, I), dtype=np.int8)).cuda()
    X[0, 0, :16] = 127               # the largest sums
    X[0, 1, :16] = -128
    _same(layer, lambda y: layer.conv2d(X, (1, 1), (0, 0), shift=shift, out=y), layer.out_shape(B, L, J, (1, 1), (0, 0)), torch.int8, torch.int8)


@pytest.mark.parametrize("dtype", ["bf16", "i8"])
@pytest.mark.parametrize("B,L,J", [(1, 300, 300), (3, 211, 210)])
def test_pixels_times_an_images_pixels_past_32_bits(dtype, B, L, J):
    """No pixel number is divided at stride 1: the kernel takes such layers, every pixel right."""
    import torch
    I, O = 64, 128
    print("large images", dtype, B, L, J, flush=True)
    rng = np.random.default_rng(O)
    gamma = _mask(O, O, I, 8, 8, 0.5)
    keep = torch.from_numpy(np.kron(gamma, np.ones((8, 8), np.uint8))).cuda()
    shape = (B, L, J, O)
    if dtype == "bf16":
        W = torch.from_numpy(rng.standard_normal((O, 1, 1, I), dtype=np.float32)).bfloat16().cuda()
        X = torch.from_numpy(rng.standard_normal((B, L, J, I), dtype=np.float32)).bfloat16().cuda()
        layer = bsp.BspLayer(W.float().cpu().numpy(), gamma, 8, 8, "bf16")
        out = torch.full(shape, float("nan"), dtype=torch.bfloat16, device="cuda")
        ran = kernels_of(lambda: layer.conv2d(X, (1, 1), (0, 0), out=out))
    else:
        W = torch.from_numpy(rng.integers(-127, 128, (O, 1, 1, I), dtype=np.int8)).cuda()
        X = torch.from_numpy(rng.integers(-128, 128, (B, L, J, I), dtype=np.int8)).cuda()
        layer = bsp.BspLayerI8(W.cpu().numpy(), gamma, 8, 8)
        out = torch.full(shape, 77, dtype=torch.int8, device="cuda")
        ran = kernels_of(lambda: layer.conv2d(X, (1, 1), (0, 0), shift=9, out=out))
    assert any("conv_pws<" in k for k in ran), ran
    want = conv_fp64(X, W * keep[:, None, None, :], 1, (0, 0))
    if dtype == "i8":  # (whole numbers below 2^53: exact)
        assert bool((out.double() == torch.floor(want / 512 + 0.5).clamp(-128, 127)).all())
        return
    scale = torch.maximum(want.abs(), want.pow(2).mean().sqrt())
    assert bool(((out.double() - want).abs() <= 6e-3 * scale).all())  # one rounding to bf16 is 3.9e-3 at most


def _instances():
    """Kind, most steps, loads a lane and residual of every instance, and a layer that runs on it: its strips and the
    16-byte pieces of its pixels."""
    cases = []
    for kind in (8, 4, 16):
        for D in (1, 2, 4, 6, 8) if kind == 16 else (2, 4, 6, 8, 12, 16):
            for QL in (1, 2) if D > 8 else (1, 2, 4):
                strips, waves = (8, 4) if D == 1 else (8, 8)
                pieces = QL * 64 * waves // (32 if D <= 8 else 16)
                if pieces < 4 * D:  # sixteen waves bring more
                    strips, pieces = 9, 2 * pieces
                cases += [(kind, D, QL, res, strips, max(pieces - 1, 4 * D)) for res in ((False,) if kind == 16 else (False, True))]
    return cases


@pytest.mark.parametrize("kind,D,QL,residual,strips,pieces", _instances())
def test_every_instance(kind, D, QL, residual, strips, pieces):
    import torch
    print("pws instance", kind, D, QL, residual, strips, pieces, flush=True)
    bo, bi = (16, 4) if kind == 4 else (8, 8)
    I, O = pieces * (16 if kind == 16 else 8), strips * 16
    rng = np.random.default_rng(D)
    units, step = (2 * pieces, 8) if kind == 4 else (pieces, 4)   # of the contraction: in all, in a step
    gamma = np.zeros((O // bo, I // bi), np.uint8)
    gamma[:, rng.permutation(units)[:D * step - 1] * (2 if kind == 16 else 1)] = 1  # every strip has the same, in D steps
    B, L, J = 1, 300 if kind == 16 and D <= 2 else 200, 181
    gen = torch.Generator("cuda").manual_seed(D)
    if kind == 16:
        layer = bsp.BspLayerI8(rng.integers(-127, 128, (O, 1, 1, I), dtype=np.int8), gamma, bo, bi, bias=rng.integers(-5000, 5001, O).astype(np.int32))
        X = torch.randint(-128, 128, (B, L, J, I), generator=gen, device="cuda", dtype=torch.int8)
        call, dtype, bits = (lambda y: layer.conv2d(X, (1, 1), (0, 0), shift=9, out=y)), torch.int8, torch.int8
    else:
        layer = bsp.BspLayer(torch.randn(O, 1, 1, I, generator=gen, device="cuda").bfloat16().float().cpu().numpy(), gamma, bo, bi, "bf16",
                             bias=rng.standard_normal(O).astype(np.float32))
        X = torch.randn(B, L, J, I, generator=gen, device="cuda").bfloat16()
        R = torch.randn(B, L, J, O, generator=gen, device="cuda").bfloat16() if residual else None
        call, dtype, bits = (lambda y: layer.conv2d(X, (1, 1), (0, 0), out=y, residual=R, relu=True)), torch.bfloat16, torch.int16
    name = "conv_pws<%d, %d, %d, %d, %d, %s>" % (kind, 2 if D <= 8 else 1, 2 if D == 1 else 1, D, QL, str(residual).lower())
    out = torch.empty((B, L, J, O), dtype=dtype, device="cuda")
    ran = kernels_of(lambda: call(out))
    assert any(name in k for k in ran), (name, ran)
    _same(layer, call, (B, L, J, O), dtype, bits)
