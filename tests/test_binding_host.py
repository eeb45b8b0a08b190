"""Marshalling of the binding that needs no GPU."""
import types

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
