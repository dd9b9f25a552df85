"""Arguments of the layer calls from Python that no device is needed for: with an empty batch a call checks
everything and launches nothing."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2407_09453_amd as bsp


class Stream:
    """What ctypes looks for in an object that stands for a C value (a torch Stream has the same)."""
    _as_parameter_ = ctypes.c_void_p(0x5000)


def _calls(stream, **args):
    rng = np.random.default_rng(0)
    gamma = np.ones((2, 2), np.uint8)
    layer = bsp.BspLayer(rng.standard_normal((16, 3, 3, 16)).astype(np.float32), gamma, 8, 8, "f32", device="cpu")
    codes = bsp.BspLayerI8(rng.integers(-9, 9, (16, 3, 3, 16)).astype(np.int8), gamma, 8, 8, device="cpu")
    fc = bsp.BspLayer(rng.standard_normal((16, 1, 1, 16)).astype(np.float32), gamma, 8, 8, "f32", device="cpu")
    fc8 = bsp.BspLayerI8(rng.integers(-9, 9, (16, 1, 1, 16)).astype(np.int8), gamma, 8, 8, device="cpu")
    X, Xq = torch.zeros(0, 5, 5, 16), torch.zeros(0, 5, 5, 16, dtype=torch.int8)
    R = torch.zeros(0, 5, 5, 16)
    return [lambda: layer.conv2d(X, pad=(1, 1), stream=stream), lambda: layer.conv2d(X, pad=(1, 1), stream=stream, residual=R, relu=True),
            lambda: fc.fc(X[:, 0, 0], stream=stream), lambda: fc.fc(X[:, 0, 0], stream=stream, relu=True),
            lambda: codes.conv2d(Xq, pad=(1, 1), stream=stream), lambda: codes.conv2d(Xq, pad=(1, 1), shift=3, stream=stream),
            lambda: fc8.fc(Xq[:, 0, 0], stream=stream), lambda: fc8.fc(Xq[:, 0, 0], shift=3, stream=stream)]


@pytest.mark.parametrize("stream", [0, 0x5000, Stream(), ctypes.c_void_p(None), ctypes.c_void_p(0x5000)],
                         ids=["null", "handle", "object", "null pointer", "pointer"])
def test_streams_that_ctypes_takes(stream):
    for call in _calls(stream):
        assert call().shape[0] == 0


@pytest.mark.parametrize("stream", [2.0, object()], ids=["float", "object"])
def test_streams_that_ctypes_refuses(stream):
    for call in _calls(stream):
        with pytest.raises(ctypes.ArgumentError):
            call()


def test_packed_calls_that_are_none():
    packed = bsp.binding.load_library().bsp_call_packed
    assert packed(0, None) == -1
    for call in (-1, 4):
        assert packed(call, bytes(14 * 8)) == -2
    for call in range(4):
        assert packed(call, bytes(14 * 8)) == -1  # no weights
