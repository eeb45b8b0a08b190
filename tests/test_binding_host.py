"""Marshalling of the binding that needs no GPU."""
import ctypes
import types

import numpy as np
import pytest

from paper_2506_19852_amd import binding as rb


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_with_and_without_the_raw_query(monkeypatch, raw):
    import torch
    monkeypatch.setattr(rb, "_current_stream", None, raising=False)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=77))
    if raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 1000 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert rb._stream_ptr(None).value == (1003 if raw else 77)
    assert rb._stream_ptr(None).value == (1003 if raw else 77)
    assert rb._stream_ptr(5).value == 5
    assert rb._stream_ptr(types.SimpleNamespace(cuda_stream=6)).value == 6


class FakeTensor:
    """As much of a CUDA tensor as the marshalling looks at."""
    is_cuda = True

    def __init__(self, dtype, *shape):
        import torch
        self.dtype, self.shape = dtype, torch.Size(shape)

    def stride(self):
        out, n = [], 1
        for d in reversed(self.shape):
            out.insert(0, n)
            n *= d
        return tuple(out)

    def is_contiguous(self):
        return True

    def dim(self):
        return len(self.shape)

    def data_ptr(self):
        return 4096

    def numel(self):
        return self.shape.numel()

    def element_size(self):
        return self.dtype.itemsize


@pytest.mark.parametrize("call", ["fwd", "trace", "fp8", "bwd", "static"])
@pytest.mark.parametrize("scale", [None, "0.5", b"1", [0.5], ctypes.c_float(0.5)])
def test_a_scale_that_is_no_number_is_a_type_error(monkeypatch, call, scale):
    """As for any wrong argument of a Python call; the library is not entered."""
    import torch
    x, lse = FakeTensor(torch.bfloat16, 1, 1, 128, 128), FakeTensor(torch.float32, 1, 1, 128)
    codes, scales = FakeTensor(torch.uint8, 1, 1, 128, 128), FakeTensor(torch.float32, 1, 1, 1)
    mask = types.SimpleNamespace(handle=None)  # the library would refuse it
    run = {"fwd": lambda: rb.radial_attn_fwd(x, x, x, x, lse, mask, scale, stream=1),
           "trace": lambda: rb.radial_attn_fwd_trace(x, x, x, x, lse, mask, scale, FakeTensor(torch.int64, 1, 3), stream=1),
           "fp8": lambda: rb.radial_attn_fwd_fp8(codes, scales, codes, scales, x, x, lse, mask, scale, stream=1),
           "bwd": lambda: rb.radial_attn_bwd(x, x, x, x, x, lse, x, x, x, mask, scale, FakeTensor(torch.uint8, 1024), stream=1),
           "static": lambda: rb.radial_attn_bwd_static(x, x, x, x, x, lse, x, x, x, mask, scale, stream=1)}[call]
    with pytest.raises(TypeError):
        run()


@pytest.mark.parametrize("scale", [1, 0.5, True, np.float32(0.5), np.float64(0.5), np.int64(1), "tensor"])
def test_a_scale_that_is_a_number_reaches_the_library(scale):
    import torch
    scale = torch.tensor(0.5) if isinstance(scale, str) else scale
    x, lse = FakeTensor(torch.bfloat16, 1, 1, 128, 128), FakeTensor(torch.float32, 1, 1, 128)
    with pytest.raises(rb.RadialError, match="mask is NULL"):
        rb.radial_attn_fwd(x, x, x, x, lse, types.SimpleNamespace(handle=None), scale, stream=1)
