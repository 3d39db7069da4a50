"""The binding asks torch for the current stream: by its raw accessors, or
through the public Stream object where a torch has none."""

from types import SimpleNamespace

import pytest
import torch

S = pytest.importorskip("paper_2606_26587_amd.sharq")


def test_stream_by_the_raw_accessors():
    c = SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda d: 100 + d)
    assert S._stream_handle(c)() == 103


@pytest.mark.parametrize("have", [{}, {"_cuda_getDevice": lambda: 0}, {"_cuda_getCurrentRawStream": lambda d: 0}])
def test_stream_without_them(monkeypatch, have):
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=77))
    assert S._stream_handle(SimpleNamespace(**have))() == 77


def test_given_stream():
    assert S._stream(SimpleNamespace(cuda_stream=5)) == 5
