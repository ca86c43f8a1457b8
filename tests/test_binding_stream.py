"""The stream a call is enqueued on: torch's current one, also where torch lacks the short way to its handle."""
import types

import torch

from paper_2402_14808_amd import binding


def test_stream_without_the_short_way(monkeypatch):
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1230))
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.delattr(torch._C, name, raising=False)
    assert binding._stream() == 0x1230
