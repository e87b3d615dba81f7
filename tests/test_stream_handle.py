"""The stream handle that the binding passes on, with torch's raw getter and
without it."""

import types

import pytest
import torch

from paper_2608_00528_amd import api


def test_torch_without_the_raw_getter(monkeypatch):
    monkeypatch.setattr(api, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=0x1234))
    assert api._stream() == 0x1234


@pytest.mark.gpu
def test_handles_agree(monkeypatch):
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            raw = api._stream()
            with monkeypatch.context() as m:
                m.setattr(api, "_raw_stream", None)
                assert api._stream() == raw == stream.cuda_stream
