"""The stream that the binding passes on: the current one, with and without torch's private lookups."""
import types

import pytest
import torch

from paper_2106_10796_amd import binding


@pytest.mark.parametrize("missing", [("_raw_stream",), ("_current_device",), ("_raw_stream", "_current_device")])
def test_falls_back_where_a_lookup_is_missing(monkeypatch, missing):
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 11)
    monkeypatch.setattr(binding, "_current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert binding._stream() == 11
    for name in missing:
        monkeypatch.setattr(binding, name, None)
    assert binding._stream() == 77


@pytest.mark.gpu
@pytest.mark.parametrize("missing", [(), ("_raw_stream",), ("_current_device",)])
def test_is_the_current_stream(monkeypatch, missing):
    torch.zeros(1, device="cuda")
    for name in missing:
        monkeypatch.setattr(binding, name, None)
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream() == side.cuda_stream
    assert binding._stream() == torch.cuda.current_stream().cuda_stream
