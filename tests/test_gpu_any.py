"""The any-shape kernel (bf16 layers with ragged channels, small layers, int8) at the sizes where
its tiles, chunks, slabs and output pieces end, against the oracle (needs a GPU)."""
import numpy as np
import pytest

import oracle
import paper_2407_09453_amd as bsp
from synthetic import draw_layer

from gpu_util import assert_close, kernels_of, make_layer, to_device, to_host

pytestmark = pytest.mark.gpu

# B, L, J, I, O, H, K, stride, pad
SHAPES = [
    (1, 1, 1, 9, 1, 1, 1, 1, 0),            # one pixel, one channel out, a chunk and a bit
    (1, 3, 5, 17, 15, 1, 1, 1, 0),          # fewer pixels than a tile, a strip that is not full
    (1, 1, 65, 130, 33, 1, 1, 1, 0),        # one pixel past four tiles, three strips
    (3, 16, 16, 40, 76, 1, 1, 2, 0),        # strided pointwise
    (2, 9, 16, 24, 40, 3, 3, 1, 1),         # rows of exactly one tile
    (1, 5, 65, 19, 9, 3, 3, 1, 1),          # rows of two chunks
    (1, 31, 63, 47, 66, 3, 3, 2, 1),
    (2, 13, 11, 70, 136, 5, 5, 1, 2),       # two slabs, the second one short
    (1, 20, 20, 33, 24, 1, 7, 2, 3),        # one-row window, strided: rows in between are not staged
    (1, 20, 20, 33, 24, 7, 1, 2, 3),
    (1, 7, 7, 512, 64, 3, 3, 1, 1),         # few pixels, long contraction: a strip shared by waves
    (1, 5, 40, 3001, 8, 5, 5, 1, 2),        # a pixel's channels staged in several pieces
    (1, 3, 3, 4101, 8, 3, 3, 1, 1),         # more slabs than the kernel takes: the general one
    (2, 50, 50, 61, 130, 3, 3, 1, 1),       # many tiles, several workgroups per tile
    (1, 6, 7, 16, 16, 3, 3, 1, 4),          # padding wider than the window
]


def _pad(H, K, p):
    return (p if H > 1 or K == 1 else 0, p if K > 1 or H == 1 else 0)


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("fused", [False, True], ids=["plain", "fused"])
def test_bf16_shapes(bo, bi, fused):
    import torch
    for n, (B, L, J, I, O, H, K, s, p) in enumerate(SHAPES):
        c = draw_layer("t", B=B, L=L, J=J, I=I, O=O, H=H, K=K, stride=(s, s), pad=_pad(H, K, p), bo=bo, bi=bi, dtype="bf16",
                       mask_kind="bernoulli", density=0.5, seed=9300 + n, b_std=0.5)
        print("case", n, SHAPES[n], bo, bi, fused, flush=True)
        layer = make_layer(c)
        Y = torch.full((c.B, c.M, c.N, c.O), float("nan"), device="cuda", dtype=torch.bfloat16)
        if not fused:
            layer.conv2d(to_device(c), c.stride, c.pad, out=Y)
            torch.cuda.synchronize()
            assert_close(to_host(Y), oracle.conv2d(c.X, c.W, c.bias, c.gamma, bo, bi, c.stride, c.pad), "bf16", f"shape {n}")
            continue
        # bit for bit the plain call followed by torch's add and relu, each rounding once
        R = torch.randn(Y.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(n)).bfloat16()
        layer.conv2d(to_device(c), c.stride, c.pad, out=Y, residual=R, relu=True)
        Y0 = layer.conv2d(to_device(c), c.stride, c.pad)
        torch.cuda.synchronize()
        assert torch.equal(Y, torch.relu(Y0.float() + R.float()).bfloat16()), n


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
def test_i8_shapes_bit_exact(bo, bi):
    import torch
    for n, (B, L, J, I, O, H, K, s, p) in enumerate(SHAPES):
        rng = np.random.default_rng(9400 + n)
        X = rng.integers(-128, 128, (B, L, J, I), dtype=np.int8)
        W = rng.integers(-128, 128, (O, H, K, I), dtype=np.int8)
        bias = rng.integers(-2 ** 18, 2 ** 18, O).astype(np.int32)
        gamma = (rng.random((-(-O // bo), -(-I // bi))) < 0.5).astype(np.uint8)
        print("case", n, SHAPES[n], bo, bi, flush=True)
        layer = bsp.BspLayerI8(W, gamma, bo, bi, bias=bias)
        # an input that starts eight bytes into its allocation, and one that is aligned
        buf = torch.zeros(X.size + 8, dtype=torch.int8, device="cuda")
        Xo = buf[8:].view(X.shape)
        Xo.copy_(torch.from_numpy(X))
        pad = _pad(H, K, p)
        Y32 = layer.conv2d(Xo, (s, s), pad)
        Y8 = layer.conv2d(torch.from_numpy(X).cuda(), (s, s), pad, shift=9)
        torch.cuda.synchronize()
        want = oracle.conv2d_i8(X, W, bias, gamma, bo, bi, (s, s), pad)
        assert (Y32.cpu().numpy().astype(np.int64) == want).all(), n
        assert (Y8.cpu().numpy() == oracle.conv2d_i8(X, W, bias, gamma, bo, bi, (s, s), pad, shift=9)).all(), n


def test_infinities_in_dropped_channels_stay_out():
    """Channels whose blocks are all dropped are never multiplied, also where a step of the plan
    has fewer pairs than a matrix instruction takes."""
    import torch
    for I, H in ((41, 3), (73, 1), (200, 3)):
        c = draw_layer("t", B=1, L=9, J=9, I=I, O=24, H=H, K=H, stride=(1, 1), pad=(H // 2, H // 2), bo=8, bi=8, dtype="bf16",
                       mask_kind="bernoulli", density=0.5, seed=9500 + I)
        c.gamma[:, 0] = 0
        c.gamma[:, -1] = 0
        X = c.X.copy()
        c.X[..., :8] = np.inf
        c.X[..., (I - 1) // 8 * 8:] = np.nan
        y = to_host(make_layer(c).conv2d(to_device(c), c.stride, c.pad))
        assert_close(y, oracle.conv2d(X, c.W, c.bias, c.gamma, 8, 8, c.stride, c.pad), "bf16", f"{I} channels")


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
def test_infinities_reach_the_rows_that_keep_their_channel_and_no_others(bo, bi):
    """An output is infinite or NaN where a kept weight meets such an input, and finite everywhere
    else: in all block rows of a strip, whatever their neighbours in it keep."""
    import torch
    for n, (B, L, J, I, O, H, K, s, p) in enumerate([
            (33, 1, 1, 64, 256, 1, 1, 1, 0), (64, 1, 1, 2048, 72, 1, 1, 1, 0), (40, 1, 1, 520, 44, 1, 1, 1, 0),
            (1, 9, 9, 41, 24, 3, 3, 1, 1), (3, 10, 15, 304, 16, 7, 1, 1, 3), (1, 8, 8, 128, 48, 3, 3, 1, 1),
            (1, 6, 6, 352, 40, 5, 5, 1, 2), (2, 14, 15, 70, 20, 5, 5, 2, 2)]):
        pad = _pad(H, K, p)
        c = draw_layer("t", B=B, L=L, J=J, I=I, O=O, H=H, K=K, stride=(s, s), pad=pad, bo=bo, bi=bi, dtype="bf16",
                       mask_kind="bernoulli", density=0.5, seed=9700 + n, b_std=0.5)
        print("case", n, (B, L, J, I, O, H, K), bo, bi, flush=True)
        conv = lambda X: oracle.conv2d(X, c.W, None, c.gamma, bo, bi, c.stride, c.pad)
        rng = np.random.default_rng(n)
        hit, X0 = {}, c.X.copy()
        for v in (np.inf, -np.inf, np.nan):
            one = np.zeros_like(c.X)
            at = rng.integers(B), rng.integers(L), rng.integers(J), rng.integers(I)
            one[at], X0[at], c.X[at] = 1.0, 0.0, v
            hit[str(v)] = conv(one)      # at most one product per output: its sign is the weight's
        up = (hit["inf"] > 0) | (hit["-inf"] < 0)
        down = (hit["inf"] < 0) | (hit["-inf"] > 0)
        nan = (hit["nan"] != 0) | (up & down)
        y = to_host(make_layer(c).conv2d(to_device(c), c.stride, c.pad))
        torch.cuda.synchronize()
        assert (np.isnan(y) == nan).all(), n
        assert (np.isposinf(y) == (up & ~nan)).all() and (np.isneginf(y) == (down & ~nan)).all(), n
        want = oracle.conv2d(X0, c.W, c.bias, c.gamma, bo, bi, c.stride, c.pad)
        ok = ~(up | down | nan)
        assert_close(np.where(ok, y, 0.0), np.where(ok, want, 0.0), "bf16", f"case {n}")


def _without(c, X):
    """The oracle's results for what the first block row keeps: an input whose infinities are zeros."""
    x = to_host(X)
    return oracle.conv2d(np.where(np.isfinite(x), x, 0.0).astype(np.float32), c.W, c.bias, c.gamma, 8, 8, c.stride, c.pad)


@pytest.mark.parametrize("B,L,J,I,O,H", [
    (1, 64, 128, 20, 64, 3), (1, 65, 128, 20, 64, 3),  # many results: through the image of the output
    (1, 50, 125, 20, 64, 3), (1, 51, 125, 20, 64, 3),  # the last and the first past the line, and the same of narrow layers
    (1, 50, 100, 20, 32, 3), (1, 51, 100, 20, 32, 3),
    (1, 9, 11, 20, 66, 3),     # few results, but a lane's four channels can end past the last one
    (1, 7, 9, 64, 16, 3),      # 1 .. 4 and 16 to 17 steps a wave: either side of the rings' ends
    (1, 5, 5, 512, 16, 3), (1, 8, 8, 1024, 36, 3), (2, 6, 6, 96, 64, 5), (4, 15, 15, 136, 24, 3),
])
def test_both_ways_out(B, L, J, I, O, H):
    """Results with bias, residual and ReLU, and an infinity in a dropped block, on both ways out of the kernel."""
    import torch
    pad = (H // 2, H // 2)
    c = draw_layer("t", B=B, L=L, J=J, I=I, O=O, H=H, K=H, stride=(1, 1), pad=pad, bo=8, bi=8, dtype="bf16", mask_kind="bernoulli", density=0.5,
                   seed=9600 + I + L, b_std=0.5)
    c.gamma[0, 1], c.gamma[1, 1] = 0, 1  # two rows of one strip: the second keeps what the first drops
    layer, X = make_layer(c), to_device(c)
    y0 = layer.conv2d(X, c.stride, c.pad)
    # the last template argument of the kernel that ran: straight from the accumulators, or through the image
    ran = [k for k in kernels_of(lambda: layer.conv2d(X, c.stride, c.pad)) if "conv_any<" in k]
    if ran:
        assert (", true>" in ran[0]) == (O % 4 == 0 and B * L * J * O <= (160000 if O < 64 else 400000)), ran
    R = torch.randn(y0.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(I)).bfloat16()
    y = layer.conv2d(X, c.stride, c.pad, residual=R, relu=True)
    torch.cuda.synchronize()
    assert_close(to_host(y0), oracle.conv2d(c.X, c.W, c.bias, c.gamma, 8, 8, c.stride, c.pad), "bf16")
    assert torch.equal(y, torch.relu(y0.float() + R.float()).bfloat16())
    X[0, 2, 3, 8:16] = float("inf")
    z = layer.conv2d(X, c.stride, c.pad)
    torch.cuda.synchronize()
    assert_close(to_host(z[..., :8]), _without(c, X)[..., :8], "bf16")
    assert not torch.isfinite(z[0, 2, 3, 8:16]).any()
    far = torch.ones(z.shape[:3], dtype=torch.bool, device="cuda")
    far[0, max(0, 2 - H // 2):3 + H // 2, max(0, 3 - H // 2):4 + H // 2] = False
    assert torch.equal(z[far], y0[far])


def test_calls_go_to_the_current_stream():
    import torch
    from paper_2407_09453_amd.binding import _current_stream
    t = torch.zeros(8, device="cuda")
    for s in (torch.cuda.current_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(s):
            assert _current_stream(t) == torch.cuda.current_stream().cuda_stream == s.cuda_stream
    with pytest.raises(ValueError):
        _current_stream(torch.zeros(8))


def test_fixed_scratch_refuses_what_it_refused():
    """The FC entry point with the fixed array: as many bits as the other, and CAPACITY by the
    documented size of the partial sums, also where a kernel without partial sums takes the layer."""
    import torch
    rng = np.random.default_rng(0)
    for O, refused in ((1000, False), (4096, True)):
        W = (rng.standard_normal((O, 1, 1, 2048)) * 0.05).astype(np.float32)
        layer = bsp.BspLayer(W, (rng.random((O // 8, 256)) < 0.5).astype(np.uint8), 8, 8, "bf16")
        X = torch.randn(64, 2048, device="cuda").bfloat16()
        Y = torch.empty(64, O, device="cuda", dtype=torch.bfloat16)
        st = torch.cuda.current_stream().cuda_stream
        call = lambda: bsp.binding.bsp_fc_fused_static(layer.struct, X.data_ptr(), None, None, False, Y.data_ptr(), 64, st)
        if refused:
            with pytest.raises(bsp.BspError) as e:
                call()
            assert e.value.code == -7
        else:
            call()
            assert torch.equal(Y, layer.fc(X))


@pytest.mark.parametrize("dtype", ("bf16", "i8"))
@pytest.mark.parametrize("O", (1, 2, 3, 4, 5, 18, 24, 35, 41))
def test_bias_of_the_last_channels(O, dtype):
    """Last strips of every remainder of four and sixteen channels: each channel gets its own bias, and
    nothing is taken from past the bias's end (a large value stands there)."""
    import torch
    rng = np.random.default_rng(O)
    B, L, I = 2, 9, 72
    nbr, nbc = -(-O // 8), -(-I // 8)
    gamma = np.ones((nbr, nbc), np.uint8)
    bias = rng.integers(-3000, 3000, O + 16).astype(np.int32 if dtype == "i8" else np.float32)
    bias[O:] = 1 << 20
    X = rng.integers(-4, 5, (B, L, L, I)).astype(np.int8)
    W = rng.integers(-3, 4, (O, 3, 3, I)).astype(np.int8)
    want = oracle.conv2d_i8(X, W, bias[:O].astype(np.int32), gamma, 8, 8, (1, 1), (1, 1), shift=None)
    if dtype == "i8":
        layer, x = bsp.BspLayerI8(W, gamma, 8, 8, bias=bias[:O]), torch.from_numpy(X).cuda()
    else:
        layer, x = bsp.BspLayer(W.astype(np.float32), gamma, 8, 8, "bf16", bias=bias[:O]), torch.from_numpy(X).cuda().bfloat16()
    layer.d_bias = torch.from_numpy(bias).cuda()
    for relu in ((False, True) if dtype == "bf16" else (False,)):
        y = layer.conv2d(x, (1, 1), (1, 1), **({"relu": relu} if dtype == "bf16" else {"shift": None}))
        torch.cuda.synchronize()
        w = torch.from_numpy(np.asarray(want)).cuda()
        if dtype == "i8":
            assert torch.equal(y, w.int())
        else:  # whole numbers below 2^24: the sums are exact and rounded once
            assert torch.equal(y, (w.relu() if relu else w).float().bfloat16())
