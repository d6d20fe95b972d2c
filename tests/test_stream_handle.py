"""The current stream's raw handle with and without torch's bare function (no GPU needed)."""
import types

import torch

from paper_2606_01478_amd import binding as B


def test_public_interface_where_the_bare_function_is_missing(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 100 + d, raising=False)
    assert B._stream() == 103
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert B._stream() == 77
