"""bsp_call_packed against the entry points that it stands for, bit for bit, with arguments that are all different
(needs a GPU)."""
import ctypes

import numpy as np
import pytest

import paper_2407_09453_amd as bsp
from paper_2407_09453_amd.binding import (BSP_CALL_CONV2D, BSP_CALL_CONV2D_I8, BSP_CALL_FC, BSP_CALL_FC_I8, BSP_I8, BSP_I32, bsp_conv2d_fused,
                                          bsp_conv2d_i8, bsp_fc_fused, bsp_fc_i8, load_library)

pytestmark = pytest.mark.gpu

B, L, J, I, O, STRIDE, PAD = 3, 17, 23, 24, 40, (2, 3), (1, 4)


def _packed(call, *words):
    a = (ctypes.c_int64 * 14)(*words)
    assert load_library().bsp_call_packed(call, ctypes.cast(a, ctypes.c_char_p)) == 0


def _weights(H, K):
    rng = np.random.default_rng(H)
    gamma = (rng.random((5, 3)) < 0.6).astype(np.uint8)
    return rng, rng.standard_normal((O, H, K, I)).astype(np.float32), gamma


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("fc", [False, True], ids=["conv", "fc"])
@pytest.mark.parametrize("fused", [False, True], ids=["plain", "fused"])
def test_floating_point_layers(dtype, fc, fused):
    import torch
    H, K = (1, 1) if fc else (3, 5)
    rng, W, gamma = _weights(H, K)
    layer = bsp.BspLayer(W, gamma, 8, 8, dtype, bias=rng.standard_normal(O).astype(np.float32))
    shape = (B * L, I) if fc else (B, L, J, I)
    X = torch.randn(shape, device="cuda").to(layer.torch_dtype)
    out = [torch.full((B * L, O) if fc else layer.out_shape(B, L, J, STRIDE, PAD), float("nan"), dtype=layer.torch_dtype, device="cuda")
           for _ in range(3)]
    R = torch.randn(out[0].shape, device="cuda").to(layer.torch_dtype) if fused else None
    r, w, b, st = (R.data_ptr() if fused else 0), layer.struct, layer.d_bias.data_ptr(), torch.cuda.current_stream().cuda_stream
    head = (ctypes.addressof(w), X.data_ptr(), b, r, int(fused))
    if fc:
        bsp_fc_fused(w, X.data_ptr(), b, r, fused, out[0].data_ptr(), B * L, st)
        _packed(BSP_CALL_FC, *head, out[1].data_ptr(), B * L, -1, -1, -1, -1, -1, -1, st)
        layer.fc(X, out=out[2], residual=R, relu=fused)
    else:
        bsp_conv2d_fused(w, X.data_ptr(), b, r, fused, out[0].data_ptr(), B, L, J, STRIDE, PAD, st)
        _packed(BSP_CALL_CONV2D, *head, out[1].data_ptr(), B, L, J, *STRIDE, *PAD, st)
        layer.conv2d(X, STRIDE, PAD, out=out[2], residual=R, relu=fused)
    assert out[0].isfinite().all() and torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])


@pytest.mark.parametrize("fc", [False, True], ids=["conv", "fc"])
@pytest.mark.parametrize("shift", [None, 0, 7])
def test_integer_layers(fc, shift):
    import torch
    H, K = (1, 1) if fc else (3, 5)
    rng, W, gamma = _weights(H, K)
    layer = bsp.BspLayerI8(bsp.bsp_quantize(W)[0], gamma, 8, 8, bias=rng.integers(-999, 999, O).astype(np.int32))
    X = torch.randint(-128, 128, (B * L, I) if fc else (B, L, J, I), dtype=torch.int8, device="cuda")
    dt, code = (torch.int32, BSP_I32) if shift is None else (torch.int8, BSP_I8)
    out = [torch.full((B * L, O) if fc else layer.out_shape(B, L, J, STRIDE, PAD), 77, dtype=dt, device="cuda") for _ in range(3)]
    w, b, st = layer.struct, layer.d_bias.data_ptr(), torch.cuda.current_stream().cuda_stream
    for k in (0, 1):
        args = X.data_ptr(), b, out[k].data_ptr(), code, shift or 0
        if fc:
            bsp_fc_i8(w, *args, B * L, st) if k == 0 else _packed(BSP_CALL_FC_I8, ctypes.addressof(w), *args, B * L, -1, -1, -1, -1, -1, -1, st)
        elif k == 0:
            bsp_conv2d_i8(w, *args, B, L, J, STRIDE, PAD, st)
        else:
            _packed(BSP_CALL_CONV2D_I8, ctypes.addressof(w), *args, B, L, J, *STRIDE, *PAD, st)
    layer.fc(X, shift=shift, out=out[2]) if fc else layer.conv2d(X, STRIDE, PAD, shift=shift, out=out[2])
    assert out[0].unique().numel() > 9 and torch.equal(out[0], out[1]) and torch.equal(out[0], out[2])
