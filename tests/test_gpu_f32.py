"""Single-precision layers through the dispatcher against the oracle at the sizes where the
kernels' tiles, chunks and slabs end (needs a GPU)."""
import numpy as np
import pytest

import oracle
from synthetic import draw_layer

from gpu_util import TOL, make_layer, to_device, to_host

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


@pytest.mark.parametrize("bo,bi", [(8, 8), (4, 16), (16, 4)])
@pytest.mark.parametrize("fused", [False, True], ids=["plain", "fused"])
def test_f32_shapes(bo, bi, fused):
    import torch
    for n, (B, L, J, I, O, H, K, s, p) in enumerate(SHAPES):
        pad = (p if H > 1 or K == 1 else 0, p if K > 1 or H == 1 else 0)
        c = draw_layer("t", B=B, L=L, J=J, I=I, O=O, H=H, K=K, stride=(s, s), pad=pad, bo=bo, bi=bi, dtype="f32",
                       mask_kind="bernoulli", density=0.5, seed=9100 + n, b_std=0.5)
        print("case", n, SHAPES[n], bo, bi, fused, flush=True)
        layer = make_layer(c)
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
