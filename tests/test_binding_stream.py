"""The stream handle a call gets when none is named (no GPU needed)."""
import types

import pytest
import torch

from paper_1708_08180_amd import binding


@pytest.mark.parametrize("raw", [True, False])
def test_current_stream_handle(monkeypatch, raw):
    # with torch's raw handle, and with a torch that has none
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x5678))
    if raw:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda dev: 0x1230 + dev, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert binding._stream_handle(None).value == (0x1233 if raw else 0x5678)
    assert binding._stream_handle(types.SimpleNamespace(cuda_stream=0x9ABC)).value == 0x9ABC
